"""The work that a user of this library has it do, as cases that can be timed.

A serving runtime calls the library once per denoising step and request batch:
whole blocks and steps on one GPU, the two halves around self-attention and the
attention itself on one GPU's share of a sequence-parallel request, the text
key/value cache once per request, the timestep modulation of a batch, and the
re-layout of a latent between two parallel layouts.  The listed cases take the
shapes of the repository's own workloads (``synth``): the image model (D 3072,
24 x 128 heads, MLP 12288), the video model (D 5120, 40 x 128 heads, MLP 13824)
and the small exact fp32 configuration, over the request classes from a 16 x 16
latent to a 720p video, with ragged batches between.

A case is a dict of plain values.  Lists are written as text: ``grids`` is one
token grid FxHxW per request, joined by ``;``, and lengths are joined by ``,``.
"""
import math

import torch

from paper_2606_13501_amd import binding as B

MODELS = {
    # hidden, heads, head_dim, mlp, rope sections, dtype
    "image": (3072, 24, 128, 12288, (0, 64, 64), torch.bfloat16),
    "video": (5120, 40, 128, 13824, (44, 42, 42), torch.bfloat16),
    "fp32_6x64": (384, 6, 64, 1536, (0, 32, 32), torch.float32),
    "fp32_4x128": (512, 4, 128, 2048, (44, 42, 42), torch.float32),
}
CHANNELS, PATCH = 16, (1, 2, 2)   # latent channels and patch of the denoising step
PATCH_LEN = CHANNELS * PATCH[0] * PATCH[1] * PATCH[2]


def listed():
    return [
        # the smallest call: a 16x16 latent through the exact fp32 configuration
        {"name": "block_tiny_fp32", "kind": "block", "model": "fp32_6x64", "grids": "1x8x8", "text": "77",
         "mod_given": False},
        # one block of a 512x512 image request (the smallest class that is served)
        {"name": "block_image_512", "kind": "block", "model": "image", "grids": "1x32x32", "text": "512",
         "mod_given": False},
        # one block of a 1024x1024 image request
        {"name": "block_image_1024", "kind": "block", "model": "image", "grids": "1x64x64", "text": "512",
         "mod_given": False},
        # a batch of image requests of mixed aspect ratios and prompt lengths, packed;
        # the modulation comes from a model-level timestep MLP
        {"name": "block_packed_images", "kind": "block", "model": "image",
         "grids": "1x32x32;1x29x37;1x48x27;1x16x24;1x40x41", "text": "512,77,231,18,400", "mod_given": True},
        # the largest call: one block of a 720p video request
        {"name": "block_video_720p", "kind": "block", "model": "video", "grids": "21x45x80", "text": "512",
         "mod_given": False},
        # a whole denoising step of a (shallow) image model on two ragged requests
        {"name": "step_image_4_blocks", "kind": "step", "model": "image", "grids": "1x32x32;1x33x49",
         "text": "512,120", "blocks": 4},
        # admission of video requests: the text keys and values of every block, once per request
        {"name": "text_kv_video_4_blocks", "kind": "text_kv", "model": "video", "text": "512,77,226", "blocks": 4},
        # self-attention of a packed batch on one GPU of eight: full lengths, an eighth of the heads
        {"name": "attention_sp8_share", "kind": "attention", "heads": 5, "q": "4096,9216,32760", "k": "",
         "q_stride": 640, "kv_stride": 640},
        # cross-attention of a 480p video to its prompt, keys and values side by side in the text cache
        {"name": "attention_cross_480p", "kind": "attention", "heads": 40, "q": "32760", "k": "512",
         "q_stride": 5120, "kv_stride": 10240},
        # the per-token halves of a block on one GPU of eight: rank 1's rows of an image and a 480p video
        {"name": "halves_sp8_share", "kind": "halves", "model": "video", "grids": "1x64x64;21x30x52",
         "text": "512,512", "degree": 8, "rank": 1},
        # the modulation vectors of a batch of requests at different timesteps
        {"name": "modulation_6_requests", "kind": "modulation", "model": "video", "requests": 6},
        # re-layout of the 720p latent between two steps, sequence-parallel degree 2 to 8
        {"name": "migrate_latent_2_to_8", "kind": "migrate", "grids": "21x45x80", "src": 2, "dst": 8},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _image_grid(rng, lo, hi):
    """A token grid of about lo..hi tokens, aspect ratio 1:2 to 2:1."""
    n, a = _log_int(rng, lo, hi), math.exp(rng.uniform(-0.69, 0.69))
    h = max(1, int(round(math.sqrt(n * a))))
    return "1x%dx%d" % (h, max(1, n // h))


def _video_grid(rng, hi):
    f, h, w = rng.randint(2, 21), rng.randint(12, 45), rng.randint(16, 80)
    while f * h * w > hi:
        f = max(1, f - 1)
        h = max(4, h - 1)
    return "%dx%dx%d" % (f, h, w)


def draw(rng):
    kind = rng.choice(["block", "block", "block", "step", "text_kv", "attention", "cross", "halves", "modulation",
                       "migrate"])
    if kind == "block":
        model = rng.choice(["image", "image", "video", "fp32_6x64", "fp32_4x128"])
        n = rng.choice([1, 1, 2, 3, rng.randint(4, 12)])
        if model.startswith("fp32"):
            grids = [_image_grid(rng, 16, 400) for _ in range(min(n, 4))]
        elif model == "image":
            grids = [_image_grid(rng, 100, 9216) for _ in range(n)]
        else:
            grids = [_video_grid(rng, 32760 // n) for _ in range(n)]
        text = [_log_int(rng, 8, 512 if not model.startswith("fp32") else 77) for _ in grids]
        return {"kind": "block", "model": model, "grids": ";".join(grids), "text": ",".join(map(str, text)),
                "mod_given": rng.random() < 0.5}
    if kind == "step":
        n = rng.randint(1, 4)
        return {"kind": "step", "model": "image", "grids": ";".join(_image_grid(rng, 100, 4096) for _ in range(n)),
                "text": ",".join(str(_log_int(rng, 8, 512)) for _ in range(n)), "blocks": rng.randint(1, 4)}
    if kind == "text_kv":
        n = rng.randint(1, 6)
        return {"kind": "text_kv", "model": rng.choice(["image", "video"]),
                "text": ",".join(str(_log_int(rng, 8, 512)) for _ in range(n)), "blocks": rng.randint(1, 6)}
    if kind == "attention":
        heads = rng.choice([3, 5, 6, 10, 12, 20])
        n = rng.randint(1, 5)
        lens = [_log_int(rng, 64, 40000 // heads if n > 2 else 80000 // heads) for _ in range(n)]
        return {"kind": "attention", "heads": heads, "q": ",".join(map(str, lens)), "k": "",
                "q_stride": heads * 128, "kv_stride": heads * 128}
    if kind == "cross":
        heads = rng.choice([24, 40])
        n = rng.randint(1, 4)
        return {"kind": "attention", "heads": heads,
                "q": ",".join(str(_log_int(rng, 256, 30000 // n)) for _ in range(n)),
                "k": ",".join(str(_log_int(rng, 8, 512)) for _ in range(n)),
                "q_stride": heads * 128, "kv_stride": heads * 256}
    if kind == "halves":
        degree = rng.choice([2, 4, 8])
        model = rng.choice(["image", "video"])
        n = rng.randint(1, 3)
        grids = [_image_grid(rng, 1024, 9216) if model == "image" else _video_grid(rng, 32760) for _ in range(n)]
        return {"kind": "halves", "model": model, "grids": ";".join(grids),
                "text": ",".join(str(_log_int(rng, 8, 512)) for _ in range(n)), "degree": degree,
                "rank": rng.randrange(degree)}
    if kind == "modulation":
        return {"kind": "modulation", "model": rng.choice(["image", "video"]), "requests": rng.randint(1, 32)}
    src, dst = rng.sample([1, 2, 3, 4, 5, 7, 8], 2)
    return {"kind": "migrate", "grids": _video_grid(rng, 75600), "src": src, "dst": dst}


# ------------------------------------------------------------------- shapes


def _grids(case):
    return [tuple(int(v) for v in g.split("x")) for g in case["grids"].split(";")]


def _ints(text):
    return [int(v) for v in text.split(",")]


def _cu(lens):
    out = [0]
    for n in lens:
        out.append(out[-1] + n)
    return out


def _shard(n, degree, rank):
    per = -(-n // degree)
    return min(n, rank * per), min(n, (rank + 1) * per)


# ------------------------------------------------------------------- inputs

# Linear weights and biases ~ N(0, 0.02^2), norm gains ~ 1 + N(0, 0.02^2),
# activations, text and latents ~ N(0, 1), timesteps ~ U[0, 1000)


class _Draw:
    def __init__(self, seed, dtype):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed * 1000003 + 13501)
        self.dtype = dtype

    def normal(self, *shape, std=1.0, mean=0.0, dtype=None):
        t = torch.empty(shape, dtype=torch.float32, device="cuda")
        return t.normal_(mean, std, generator=self.g).to(dtype or self.dtype)

    def uniform(self, n, lo, hi):
        return torch.empty(n, dtype=torch.float32, device="cuda").uniform_(lo, hi, generator=self.g)

    def lin(self, n_out, n_in):
        return self.normal(n_out, n_in, std=0.02)

    def bias(self, n):
        return self.normal(n, std=0.02)

    def gain(self, n):
        return self.normal(n, std=0.02, mean=1.0)


def _block_weights(r, model, tmlp=True, ada=True):
    D, H, d, Dff, _, _ = MODELS[model]
    w = {}
    if tmlp:
        w.update(w_t1=r.lin(D, D), b_t1=r.bias(D), w_t2=r.lin(D, D), b_t2=r.bias(D))
    if ada:
        w.update(w_ada=r.lin(6 * D, D), b_ada=r.bias(6 * D))
    w.update(w_qkv=r.lin(3 * D, D), b_qkv=r.bias(3 * D), g_q=r.gain(d), g_k=r.gain(d),
             w_o=r.lin(D, D), b_o=r.bias(D), g_ca=r.gain(D), b_ca=r.bias(D), w_cq=r.lin(D, D), b_cq=r.bias(D),
             w_ckv=r.lin(2 * D, D), b_ckv=r.bias(2 * D), g_cq=r.gain(d), g_ck=r.gain(d),
             w_co=r.lin(D, D), b_co=r.bias(D), w_up=r.lin(Dff, D), b_up=r.bias(Dff),
             w_dn=r.lin(D, Dff), b_dn=r.bias(D))
    return w


def _inputs(case, seed):
    """The tensors of a case, the same for prepare() and exact()."""
    kind = case["kind"]
    i = {}
    if kind == "attention":
        r = _Draw(seed, torch.bfloat16)
        h, nq = case["heads"], sum(_ints(case["q"]))
        nk = sum(_ints(case["k"])) if case["k"] else nq
        i["q"] = r.normal(nq, case["q_stride"])
        if case["kv_stride"] == 2 * h * 128:      # [k | v] side by side in one row
            i["kv"] = r.normal(nk, case["kv_stride"])
            i["k"], i["v"] = i["kv"][:, :h * 128], i["kv"][:, h * 128:]
        else:
            i["k"], i["v"] = r.normal(nk, case["kv_stride"]), r.normal(nk, case["kv_stride"])
        return i
    if kind == "migrate":
        r = _Draw(seed, torch.float32)
        F, H, W = _grids(case)[0]
        i["latent"] = r.normal(CHANNELS, F, 2 * H, 2 * W)
        return i
    D, H, d, Dff, _, dtype = MODELS[case["model"]]
    r = _Draw(seed, dtype)
    if kind == "modulation":
        i["w"] = dict(w_t1=r.lin(D, D), b_t1=r.bias(D), w_t2=r.lin(D, D), b_t2=r.bias(D),
                      w_ada=r.lin(6 * D, D), b_ada=r.bias(6 * D))
        i["t"] = r.uniform(case["requests"], 0.0, 1000.0)
        return i
    text = _ints(case["text"])
    i["txt"] = r.normal(sum(text), D)
    if kind == "text_kv":
        i["blocks"] = [dict(w_ckv=r.lin(2 * D, D), b_ckv=r.bias(2 * D), g_ck=r.gain(d))
                       for _ in range(case["blocks"])]
        return i
    grids = _grids(case)
    rows = [f * h * w for f, h, w in grids]
    if kind == "step":
        i["model"] = dict(w_t1=r.lin(D, D), b_t1=r.bias(D), w_t2=r.lin(D, D), b_t2=r.bias(D),
                          w_pe=r.lin(D, PATCH_LEN), b_pe=r.bias(D), w_hmod=r.lin(2 * D, D), b_hmod=r.bias(2 * D),
                          w_out=r.lin(PATCH_LEN, D), b_out=r.bias(PATCH_LEN))
        i["blocks"] = [_block_weights(r, case["model"], tmlp=False) for _ in range(case["blocks"])]
        i["latent"] = r.normal(sum(rows) * PATCH_LEN, dtype=torch.float32)
        i["t"] = r.uniform(len(rows), 0.0, 1000.0)
        i["dt"] = r.uniform(len(rows), -0.05, -0.01)
        return i
    if kind == "halves":
        spans = [_shard(n, case["degree"], case["rank"]) for n in rows]
        rows = [b - a for a, b in spans]
        i["offsets"] = [a for a, _ in spans]
        i["o"] = r.normal(sum(rows), D, std=0.1)   # the attention output: an average of values
    i["rows"] = rows
    i["x"] = r.normal(sum(rows), D)
    given = case.get("mod_given", False)
    i["w"] = _block_weights(r, case["model"], tmlp=not given, ada=not given)
    if given:
        i["mod"] = r.normal(len(rows), 6, D, std=0.5, dtype=torch.float32)
    else:
        i["t"] = r.uniform(len(rows), 0.0, 1000.0)
    return i


def _bytes(n):
    return torch.empty(n, dtype=torch.uint8, device="cuda")


def _config(model):
    D, H, d, Dff, rope, dtype = MODELS[model]
    return B.BlockConfig(D, H, d, Dff, D, rope, dtype)


def prepare(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    s["kind"] = kind
    if kind == "attention":
        s["heads"] = case["heads"]
        s["cu_q"] = _cu(_ints(case["q"]))
        s["cu_k"] = _cu(_ints(case["k"])) if case["k"] else s["cu_q"]
        s["o"] = torch.empty(s["q"].shape[0], case["heads"] * 128, dtype=torch.bfloat16, device="cuda")
        return s
    if kind == "migrate":
        F, H, W = _grids(case)[0]
        shape = (CHANNELS, F, 2 * H, 2 * W)

        def bands(n):
            # frames x rows of the latent, split by rows of height
            cut = [2 * H * k // n for k in range(n + 1)]
            return [(k, (0, 0, cut[k], 0), (CHANNELS, F, cut[k + 1], 2 * W)) for k in range(n)]

        src, dst = bands(case["src"]), bands(case["dst"])
        s["field"] = B.MigField(B.MIG_SHARDED, shape, 4, src, dst)
        s["entries"], s["n"] = B.migration_plan(s["field"])
        s["src"] = [s["latent"][:, :, a[2]:b[2]].contiguous() for _, a, b in src]
        s["dst"] = [torch.empty(CHANNELS, F, b[2] - a[2], 2 * W, device="cuda") for _, a, b in dst]
        return s
    D = MODELS[case["model"]][0]
    dtype = MODELS[case["model"]][5]
    cfg = s["cfg"] = _config(case["model"])
    if kind == "modulation":
        n = case["requests"]
        s["weights"] = B.make_weights(s["w"])
        s["mod"] = torch.empty(n, 6, D, device="cuda")
        s["ws"] = _bytes(4 * 3 * n * D + 1024)
        return s
    text = _ints(case["text"])
    if kind == "text_kv":
        s["mcfg"] = B.ModelConfig(cfg, case["blocks"], CHANNELS, PATCH)
        s["mw"] = B.ModelWeights({}, [B.make_weights(w) for w in s["blocks"]])
        s["vl"] = B.Varlen([0] * (len(text) + 1), _cu(text), [(1, 1, 1)] * len(text))
        s["kv"] = torch.empty(B.text_kv_elems(s["mcfg"], s["vl"]), dtype=dtype, device="cuda")
        return s
    grids = _grids(case)
    if kind == "step":
        s["mcfg"] = B.ModelConfig(cfg, case["blocks"], CHANNELS, PATCH)
        s["mw"] = B.ModelWeights(s["model"], [B.make_weights(w) for w in s["blocks"]])
        vl = s["vl"] = B.Varlen(_cu([f * h * w for f, h, w in grids]), _cu(text), grids)
        s["kv"] = torch.empty(B.text_kv_elems(s["mcfg"], vl), dtype=dtype, device="cuda")
        B.text_kv(s["mcfg"], s["mw"], vl, s["txt"], s["kv"])
        s["ws"] = _bytes(B.denoise_workspace_size(s["mcfg"], vl))
        s["next"] = torch.empty_like(s["latent"])
        return s
    s["weights"] = B.make_weights(s["w"])
    vl = s["vl"] = B.Varlen(_cu(s["rows"]), _cu(text), grids, s.get("offsets"))
    s["ws"] = _bytes(B.block_workspace_size(cfg, vl))
    s["y"] = torch.empty_like(s["x"])
    if kind == "halves":
        s["mod"] = torch.empty(len(grids), 6, D, device="cuda")
        s["qkv"] = torch.empty(3, s["x"].shape[0], D, dtype=dtype, device="cuda")
    return s


def run(s):
    kind = s["kind"]
    if kind == "block":
        B.block_forward(s["cfg"], s["weights"], s["vl"], s["x"], s.get("t"), s["txt"], s["y"], s["ws"],
                        mod=s.get("mod"))
        return s["y"]
    if kind == "halves":
        B.block_pre_attention(s["cfg"], s["weights"], s["vl"], s["x"], s["t"], s["mod"], s["qkv"], s["ws"])
        B.block_post_attention(s["cfg"], s["weights"], s["vl"], s["x"], s["o"], s["txt"], s["mod"], s["y"], s["ws"])
        return {"qkv": s["qkv"], "mod": s["mod"], "y": s["y"]}
    if kind == "step":
        B.denoise_step(s["mcfg"], s["mw"], s["vl"], s["latent"], s["t"], s["dt"], s["kv"], s["next"], s["ws"])
        return s["next"]
    if kind == "text_kv":
        B.text_kv(s["mcfg"], s["mw"], s["vl"], s["txt"], s["kv"])
        return s["kv"]
    if kind == "attention":
        B.attention_varlen(s["q"], s["k"], s["v"], s["o"], s["cu_q"], s["cu_k"], s["heads"], 128)
        return s["o"]
    if kind == "modulation":
        B.timestep_modulation(s["cfg"], s["weights"], s["t"], s["mod"], s["ws"])
        return s["mod"]
    B.migration_execute(s["field"], s["entries"], s["n"], s["src"], s["dst"])
    return s["dst"]


# --------------------------------------------------------------------- work


def _block_work(case, rows, attn_rows, text, halves=False, cond=True, text_proj=True):
    """(bytes, flops) of one block: weights, x, text and y once; no intermediate tensors."""
    D, H, d, Dff, _, dtype = MODELS[case["model"]]
    es = 2 if dtype == torch.bfloat16 else 4
    T, L, R = sum(rows), sum(text), len(rows)
    weights = D * 3 * D + 3 * D * D + 2 * D * Dff
    flops = 2 * T * weights + 4 * D * sum(a * b for a, b in zip(rows, text))
    byt = es * (weights + 2 * T * D)
    if text_proj:
        flops += 4 * L * D * D
        byt += es * (2 * D * D + L * D)
    else:
        byt += es * 2 * L * D
    if cond:
        flops += 2 * R * 6 * D * D
        byt += es * 6 * D * D
    if halves:
        byt += es * 4 * T * D          # q, k, v written, o read
    else:
        flops += 4 * D * sum(a * b for a, b in zip(rows, attn_rows))
    return byt, flops


def work(case):
    kind = case["kind"]
    if kind == "attention":
        q = _ints(case["q"])
        k = _ints(case["k"]) if case["k"] else q
        width = case["heads"] * 128
        return {"bytes": 2 * width * (2 * sum(q) + 2 * sum(k)), "flops": 4 * width * sum(a * b for a, b in zip(q, k))}
    if kind == "migrate":
        F, H, W = _grids(case)[0]
        return {"bytes": 2 * 4 * CHANNELS * F * 4 * H * W, "flops": 0}
    D = MODELS[case["model"]][0]
    es = 2 if MODELS[case["model"]][5] == torch.bfloat16 else 4
    if kind == "modulation":
        R = case["requests"]
        return {"bytes": es * 8 * D * D + 4 * R * (1 + 6 * D), "flops": 2 * R * 8 * D * D}
    text = _ints(case["text"])
    if kind == "text_kv":
        n, L = case["blocks"], sum(text)
        return {"bytes": es * (n * (2 * D * D + 2 * L * D) + L * D), "flops": n * 4 * L * D * D}
    rows = [f * h * w for f, h, w in _grids(case)]
    if kind == "step":
        n, T = case["blocks"], sum(rows)
        b, f = _block_work(case, rows, rows, text, text_proj=False)
        b -= es * 2 * T * D
        return {"bytes": n * b + 8 * T * PATCH_LEN + es * (2 * D * PATCH_LEN + 4 * D * D),
                "flops": n * f + 4 * T * D * PATCH_LEN + 2 * len(rows) * 4 * D * D}
    if kind == "halves":
        rows = [b - a for a, b in (_shard(n, case["degree"], case["rank"]) for n in rows)]
        b, f = _block_work(case, rows, rows, text, halves=True)
        return {"bytes": b + es * 2 * D * D, "flops": f + 4 * len(rows) * D * D}
    b, f = _block_work(case, rows, rows, text, cond=not case["mod_given"])
    if case["mod_given"]:
        return {"bytes": b + 4 * 6 * D * len(rows), "flops": f}
    return {"bytes": b + es * 2 * D * D, "flops": f + 4 * len(rows) * D * D}


def tolerance(case):
    """Relative error between two correct implementations at the same precision,
    about four times the distance from float64 that was measured.

    bf16: every stage of a block rounds its output to bf16 (2^-9 per value):
    1.9e-3 to 3.7e-3 on blocks, halves, attention and the text cache.  The
    step's latent is fp32 and the update a small part of it (2e-4).  fp32:
    sums in another order (blocks 2e-7, modulation 3e-7).  A re-layout moves
    bytes.
    """
    kind = case["kind"]
    if kind == "migrate":
        return "exact"
    if kind == "modulation":
        return {"rel": 1.5e-6}
    if case.get("model", "").startswith("fp32"):
        return {"rel": 1e-6}
    if kind == "step":
        return {"rel": 1e-3}
    return {"rel": 1e-2}


# -------------------------------------------------------------------- exact


def _dbl(w):
    return {k: v.double() for k, v in w.items()}


def _ln(x, eps=1e-6):
    x = x - x.mean(-1, keepdim=True)
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps)


def _rms(x, gain, d, eps=1e-6):
    h = x.view(x.shape[0], -1, d)
    return (h / torch.sqrt((h * h).mean(-1, keepdim=True) + eps) * gain).view(x.shape)


def _silu(x):
    return x / (1 + torch.exp(-x))


def _timestep(t, w, D):
    half = D // 2
    f = torch.exp(-math.log(10000.0) * torch.arange(half, device="cuda", dtype=torch.float64) / half)
    a = t.double()[:, None] * f
    e = torch.cat([torch.cos(a), torch.sin(a)], 1)
    a1 = _silu(e @ w["w_t1"].T + w["b_t1"])
    return _silu(a1 @ w["w_t2"].T + w["b_t2"])


def _sdpa(q, k, v, heads, d):
    """Softmax attention of one request, head by head, in chunks of queries."""
    o = torch.empty_like(q)
    for h in range(heads):
        c = slice(h * d, (h + 1) * d)
        kt, vh = k[:, c].T.contiguous(), v[:, c].contiguous()
        step = max(1, (1 << 29) // max(1, k.shape[0]))
        for a in range(0, q.shape[0], step):
            s = (q[a:a + step, c].contiguous() @ kt).mul_(1 / math.sqrt(d))
            s.sub_(s.amax(-1, keepdim=True)).exp_()
            o[a:a + step, c] = (s @ vh).div_(s.sum(-1, keepdim=True))
    return o


def _packed_sdpa(q, k, v, cu_q, cu_k, heads, d):
    return torch.cat([_sdpa(q[a:b], k[e:f], v[e:f], heads, d)
                      for a, b, e, f in zip(cu_q, cu_q[1:], cu_k, cu_k[1:])])


def _rope(x, grids, offsets, rows, sections, d):
    parts, at = [], 0
    for (F, H, W), off, n in zip(grids, offsets, rows):
        g = torch.arange(off, off + n, device="cuda")
        pos = [g // (H * W), (g // W) % H, g % W]
        ang = []
        for p, ds in zip(pos, sections):
            if ds:
                f = 10000.0 ** (-2.0 * torch.arange(ds // 2, device="cuda", dtype=torch.float64) / ds)
                ang.append(p.double()[:, None] * f)
        a = torch.cat(ang, 1)[:, None, :]
        h = x[at:at + n].view(n, -1, d // 2, 2)
        re, im = h[..., 0], h[..., 1]
        c, s = torch.cos(a), torch.sin(a)
        parts.append(torch.stack([re * c - im * s, re * s + im * c], -1).reshape(n, -1))
        at += n
    return torch.cat(parts)


def _per_row(v, rows):
    return torch.cat([v[r:r + 1].expand(n, -1) for r, n in enumerate(rows)])


def _pre(x, w, mod, model, grids, offsets, rows):
    D, H, d, _, sec, _ = MODELS[model]
    h = _ln(x) * (1 + _per_row(mod[:, 1], rows)) + _per_row(mod[:, 0], rows)
    q, k, v = ((h @ w["w_qkv"][i * D:(i + 1) * D].T) + w["b_qkv"][i * D:(i + 1) * D] for i in range(3))
    return (_rope(_rms(q, w["g_q"], d), grids, offsets, rows, sec, d),
            _rope(_rms(k, w["g_k"], d), grids, offsets, rows, sec, d), v)


def _post(x, o, w, mod, model, rows, txt, text):
    D, H, d, _, _, _ = MODELS[model]
    x1 = x + _per_row(mod[:, 2], rows) * (o @ w["w_o"].T + w["b_o"])
    hc = _ln(x1) * w["g_ca"] + w["b_ca"]
    cq = _rms(hc @ w["w_cq"].T + w["b_cq"], w["g_cq"], d)
    ckv = txt @ w["w_ckv"].T + w["b_ckv"]
    ck, cv = _rms(ckv[:, :D].contiguous(), w["g_ck"], d), ckv[:, D:]
    oc = _packed_sdpa(cq, ck, cv, _cu(rows), _cu(text), H, d)
    x2 = x1 + oc @ w["w_co"].T + w["b_co"]
    h2 = _ln(x2) * (1 + _per_row(mod[:, 4], rows)) + _per_row(mod[:, 3], rows)
    u = h2 @ w["w_up"].T + w["b_up"]
    u = 0.5 * u * (1 + torch.tanh(math.sqrt(2 / math.pi) * (u + 0.044715 * u ** 3)))
    return x2 + _per_row(mod[:, 5], rows) * (u @ w["w_dn"].T + w["b_dn"])


def _tokens(latent, grids, inverse=False):
    """Packed latents to patch vectors [tokens, P], or back."""
    out, at = [], 0
    pt, ph, pw = PATCH
    for F, H, W in grids:
        n = F * H * W
        if inverse:
            t = latent[at:at + n].view(F, H, W, CHANNELS, pt, ph, pw).permute(3, 0, 4, 1, 5, 2, 6)
            out.append(t.reshape(-1))
            at += n
        else:
            t = latent[at:at + n * PATCH_LEN].view(CHANNELS, F, pt, H, ph, W, pw).permute(1, 3, 5, 0, 2, 4, 6)
            out.append(t.reshape(n, PATCH_LEN))
            at += n * PATCH_LEN
    return torch.cat(out)


def exact(case, seed):
    i = _inputs(case, seed)
    kind = case["kind"]
    if kind == "attention":
        cu_q = _cu(_ints(case["q"]))
        cu_k = _cu(_ints(case["k"])) if case["k"] else cu_q
        return _packed_sdpa(i["q"].double(), i["k"].double(), i["v"].double(), cu_q, cu_k, case["heads"], 128)
    if kind == "migrate":
        H = _grids(case)[0][1]
        cut = [2 * H * k // case["dst"] for k in range(case["dst"] + 1)]
        return [i["latent"][:, :, a:b].contiguous() for a, b in zip(cut, cut[1:])]
    D, H, d, Dff, _, _ = MODELS[case["model"]]
    if kind == "modulation":
        w = _dbl(i["w"])
        return (_timestep(i["t"], w, D) @ w["w_ada"].T + w["b_ada"]).view(-1, 6, D)
    text = _ints(case["text"])
    txt = i["txt"].double()
    if kind == "text_kv":
        out = []
        for w in map(_dbl, i["blocks"]):
            kv = txt @ w["w_ckv"].T + w["b_ckv"]
            out.append(torch.cat([_rms(kv[:, :D].contiguous(), w["g_ck"], d), kv[:, D:]], 1).reshape(-1))
        return torch.cat(out)
    grids = _grids(case)
    if kind == "step":
        rows = [f * h * w for f, h, w in grids]
        m = _dbl(i["model"])
        x = _tokens(i["latent"].double(), grids) @ m["w_pe"].T + m["b_pe"]
        c = _timestep(i["t"], m, D)
        zero = [0] * len(rows)
        for w in map(_dbl, i["blocks"]):
            mod = (c @ w["w_ada"].T + w["b_ada"]).view(-1, 6, D)
            q, k, v = _pre(x, w, mod, case["model"], grids, zero, rows)
            o = _packed_sdpa(q, k, v, _cu(rows), _cu(rows), H, d)
            x = _post(x, o, w, mod, case["model"], rows, txt, text)
        hm = (c @ m["w_hmod"].T + m["b_hmod"]).view(-1, 2, D)
        v = (_ln(x) * (1 + _per_row(hm[:, 1], rows)) + _per_row(hm[:, 0], rows)) @ m["w_out"].T + m["b_out"]
        dt = torch.cat([i["dt"][r:r + 1].double().expand(n * PATCH_LEN) for r, n in enumerate(rows)])
        return i["latent"].double() + dt * _tokens(v, grids, inverse=True)
    rows = i["rows"]
    offsets = i.get("offsets", [0] * len(rows))
    w = _dbl(i["w"])
    x = i["x"].double()
    if "mod" in i:
        mod = i["mod"].double()
    else:
        mod = (_timestep(i["t"], w, D) @ w["w_ada"].T + w["b_ada"]).view(-1, 6, D)
    q, k, v = _pre(x, w, mod, case["model"], grids, offsets, rows)
    if kind == "halves":
        y = _post(x, i["o"].double(), w, mod, case["model"], rows, txt, text)
        return {"qkv": torch.stack([q, k, v]), "mod": mod, "y": y}
    o = _packed_sdpa(q, k, v, _cu(rows), _cu(rows), H, d)
    del q, k, v
    return _post(x, o, w, mod, case["model"], rows, txt, text)
