"""Workloads by which the speed of this library is judged: what a program that
holds a mixed-policy KV cache has it do, from one step of a tiny cache to a
denoising step of eight images.

Every case goes through the public entry points (the functions of the package,
`AttendPlan`, `runner.Run`).  Shapes come from the repository's own workloads
(28 query heads on 4 KV heads, head dim 128, 4096 tokens per image; the tiny
one with head dim 64 in fp32); draw() spreads them over the ranges that the
tests cover: other head counts and groups, head dim 64, fp16 and fp32, 2/4/8
bit codes, groups 8 to 128, ragged row counts.

Inputs: N(0,1) keys, values and queries with two outlier key channels (x8),
and for the long contexts a heavy-tailed rank-one term on the keys with a
matching direction in the queries, so that a few tokens dominate.
"""
import math

import numpy as np
import torch

import paper_2609_32831_amd as uc
import workloads
from paper_2609_32831_amd.runner import Run

DT = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
SIZE = {"f32": 4, "f16": 2, "bf16": 2}


# ---------------------------------------------------------------- the cases

def listed():
    head = {"Hq": 28, "Hkv": 4, "D": 128, "dtype": "bf16"}
    return [
        # a whole small request in fp32: score, evict, quantise, one decode step (latency and launches count)
        {"name": "tiny_request", "kind": "request", "text": 64, "vit": 256, "vae": 256, "W": 16, "ratio": 0.2,
         "bits": 4, "group": 32},
        # sixteen consecutive decode steps of a visual question (four requests) on an execution plan
        {"name": "understanding_steps", "kind": "decode", "api": "plan", **head, "B": 4, "M": 1, "steps": 16, "keep": 512,
         "kept": 406, "pack": 0, "bits": 4, "group": 64, "tail": 120, "capacity": 256, "heavy": 0},
        # one user with a compressed 64k context: a single decode step
        {"name": "single_64k_step", "kind": "decode", "api": "append", **head, "B": 1, "M": 1, "steps": 1, "keep": 0,
         "kept": 11735, "pack": 4096, "bits": 4, "group": 64, "tail": 300, "capacity": 512, "heavy": 1},
        # the same for a batch of sixteen: the step that long-context serving repeats
        {"name": "batch16_64k_step", "kind": "decode", "api": "append", **head, "B": 16, "M": 1, "steps": 1, "keep": 0,
         "kept": 11735, "pack": 4096, "bits": 4, "group": 64, "tail": 256, "capacity": 512, "heavy": 1},
        # sixteen requests of different lengths decoded in one call
        {"name": "mixed_batch_step", "kind": "batch", **head, "R": 16, "M": 1, "kept_min": 2000, "kept_max": 12500, "pack": 4096,
         "bits": 4, "group": 64, "tail": 9},
        # a decode step of an fp16 cache whose image rows are held in 8 bits
        {"name": "f16_8bit_step", "kind": "decode", "api": "append", "Hq": 28, "Hkv": 4, "D": 128, "dtype": "f16", "B": 4, "M": 1,
         "steps": 1, "keep": 512, "kept": 0, "pack": 4096, "bits": 8, "group": 32, "tail": 64, "capacity": 256,
         "heavy": 0},
        # a user's next prompt (about two hundred tokens) over one request's compressed editing context
        {"name": "prompt_prefill", "kind": "prefill", **head, "B": 1, "M": 203, "keep": 1024, "kept": 1024, "pack": 4096,
         "bits": 4, "group": 64, "stats": 0},
        # one denoising timestep of image editing: 4096 queries per request over text, kept ViT and int4 VAE rows
        {"name": "editing_prefill", "kind": "prefill", **head, "B": 2, "M": 4096, "keep": 1024, "kept": 1024, "pack": 4096,
         "bits": 4, "group": 64, "stats": 0},
        # one text-to-image timestep of eight images: the drifted latent re-quantised (int2/int4 by head), attended
        # with per-segment statistics, and the type masses the next widths come from
        {"name": "text_to_image_step", "kind": "denoise", **head, "B": 8, "M": 4096, "text": 768, "latent": 4096,
         "group": 64},
        # importance scores of a 64k context from a 32-row observation window, sixteen requests
        {"name": "score_64k", "kind": "score", **head, "B": 16, "W": 32, "text": 4096, "vit": 61440, "pack": 0,
         "bits": 4, "group": 64, "columns": 0, "heavy": 1},
        # importance scores of an editing context from all 4096 queries of a timestep, two requests
        {"name": "score_editing", "kind": "score", **head, "B": 2, "W": 4096, "text": 5120, "vit": 4096, "pack": 0,
         "bits": 4, "group": 64, "columns": 0, "heavy": 0},
        # the compression itself: top-k with compaction of the ViT rows and int4 codes of the text rows
        {"name": "compress_64k", "kind": "compress", **head, "B": 16, "rows": 61440, "k": 11735, "recent": 0, "quant": 4096,
         "bits": 4, "group": 64},
    ]


def spread(rng, lo, hi):
    """A whole number between lo and hi, even over its logarithm; odd ones among them."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def some_heads(rng):
    """Query heads, KV heads, head dim and element type of a model."""
    Hkv = rng.choice([1, 2, 4, 4, 8])
    G = rng.choice([1, 2, 4, 7, 7, 8, 16])
    D, dtype = rng.choice([(128, "bf16")] * 7 + [(64, "bf16"), (128, "f16"), (64, "f32")])
    return {"Hq": G * Hkv, "Hkv": Hkv, "D": D, "dtype": dtype}


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "batch", "prefill", "prefill", "denoise", "score", "score",
                       "compress", "request"])
    if kind == "request":
        return {"kind": kind, "text": spread(rng, 16, 256), "vit": spread(rng, 64, 1024), "vae": spread(rng, 32, 1024),
                "W": spread(rng, 1, 32), "ratio": round(rng.uniform(0.05, 0.9), 2), "bits": rng.choice([2, 4, 8]),
                "group": rng.choice([8, 16, 32, 64])}
    h = some_heads(rng)
    G = h["Hq"] // h["Hkv"]
    fast = h["D"] == 128 and h["dtype"] == "bf16"
    bits, group = rng.choice([2, 4, 4, 4, 8]), rng.choice([32, 64, 64] + ([128] if h["D"] == 128 else [16]))
    if kind == "decode":
        B = spread(rng, 1, 16)
        c = {"kind": kind, "api": rng.choice(["append", "append", "plan", "stream"]), **h, "B": B, "M": 1, "steps": 1,
             "keep": rng.choice([0, spread(rng, 16, 4096)]), "kept": spread(rng, 16, 12000 if fast else 2000),
             "pack": rng.choice([0, spread(rng, 64, 8192 if fast else 2048)]), "bits": bits, "group": group,
             "tail": spread(rng, 1, 500), "capacity": 516, "heavy": rng.choice([0, 1])}
        if c["api"] == "plan":
            c["steps"] = spread(rng, 1, 16)
        elif c["api"] == "stream":
            c["pack"] = c["pack"] or spread(rng, 64, 2048)
            c["steps"] = rng.choice([1, 8])
        elif G <= 8:
            c["M"] = rng.choice([1, 1, 2])
        return c
    if kind == "batch":
        return {"kind": kind, **{**h, "D": 128, "dtype": "bf16"}, "R": spread(rng, 2, 40), "M": 1,
                "kept_min": spread(rng, 16, 1000), "kept_max": spread(rng, 1000, 9000),
                "pack": rng.choice([0, spread(rng, 64, 4096)]), "bits": rng.choice([2, 4]), "group": max(32, group),
                "tail": spread(rng, 1, 300)}
    if kind == "prefill":
        c = {"kind": kind, **h, "B": spread(rng, 1, 4), "M": spread(rng, 17, 4096 if fast else 64),
             "keep": spread(rng, 16, 2048), "kept": rng.choice([0, spread(rng, 16, 4096)]),
             "pack": rng.choice([0, spread(rng, 64, 4096)]), "bits": bits, "group": group, "stats": rng.choice([0, 1])}
        n = c["keep"] + c["kept"] + c["pack"]
        most = 3e9 if fast else 3e7  # query rows x key rows x heads
        while c["B"] * h["Hq"] * c["M"] * n > most:
            c["M"] = max(1, c["M"] // 2) if c["M"] > 17 or c["B"] == 1 else c["M"]
            c["B"] = max(1, c["B"] // 2)
        return c
    if kind == "denoise":
        h = {**h, "D": 128, "dtype": "bf16"}
        c = {"kind": kind, **h, "B": spread(rng, 1, 8), "M": spread(rng, 64, 4096), "text": spread(rng, 16, 1024),
             "latent": spread(rng, 256, 4096), "group": rng.choice([32, 64, 128])}
        while c["B"] * h["Hq"] * c["M"] * (c["text"] + c["latent"]) > 3e9:
            c["B"] = max(1, c["B"] - 1)
            c["M"] = c["M"] * 3 // 4
        return c
    if kind == "score":
        W = rng.choice([spread(rng, 1, 64), spread(rng, 64, 4096)])
        c = {"kind": kind, **h, "B": spread(rng, 1, 8), "W": W, "text": spread(rng, 64, 4096),
             "vit": spread(rng, 256, 32768), "pack": rng.choice([0, 0, spread(rng, 128, 4096)]), "bits": bits,
             "group": group, "columns": rng.choice([0, 0, 1]), "heavy": rng.choice([0, 1])}
        most = 2e9 if fast else 3e7
        while c["B"] * h["Hq"] * c["W"] * (c["text"] + c["vit"] + c["pack"]) > most:
            c["B"] = max(1, c["B"] // 2)
            c["W"] = max(1, c["W"] // 2)
            c["vit"] = max(256, c["vit"] * 3 // 4)
        return c
    rows = spread(rng, 256, 65536)
    k = max(1, int(rows * rng.uniform(0.02, 0.6)))
    return {"kind": kind, **h, "B": spread(rng, 1, 8), "rows": rows, "k": k, "recent": rng.choice([0, 0, min(k, 32)]),
            "quant": spread(rng, 64, 4096), "bits": bits, "group": group}


# ---------------------------------------------------------------- inputs

def scale_of(D):
    return float(np.float32(1.0 / math.sqrt(D)))


class Source:
    """Seeded tensors on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(self, *shape):
        return torch.randn(*shape, generator=self.g, device="cuda")

    def student(self, *shape):
        """Student-t with three degrees of freedom."""
        z = self.normal(*shape)
        return z / (self.normal(*shape, 3).square().sum(-1) / 3).sqrt()


class Heads:
    """What the keys and queries of one case have in common: each KV head's
    outlier channels and (heavy) the direction its dominant keys share."""

    def __init__(self, src, c, heavy):
        B, Hkv, D = c.get("B", c.get("R")), c["Hkv"], c["D"]
        self.c, self.src, self.heavy = c, src, heavy
        self.scale = torch.ones(B, Hkv, 1, D, device="cuda")
        pick = torch.rand(B, Hkv, 1, D, generator=src.g, device="cuda").argsort(-1)[..., :2]
        self.scale.scatter_(-1, pick, 8.0)
        u = src.normal(B, Hkv, 1, D)
        self.u = u / u.norm(dim=-1, keepdim=True)

    def kv(self, n, heavy=False, b=None):
        """K and V rows [B, Hkv, n, D] of one segment (b: of one request)."""
        pick = slice(None) if b is None else slice(b, b + 1)
        s, u = self.scale[pick], self.u[pick]
        B, Hkv, D = s.shape[0], s.shape[1], s.shape[3]
        dt = DT[self.c["dtype"]]
        k = self.src.normal(B, Hkv, n, D).mul_(s)
        if heavy:
            k.addcmul_(self.src.student(B, Hkv, n, 1) * (math.sqrt(D) / 2), u)
        k = k.to(dt)
        return k, self.src.normal(B, Hkv, n, D).to(dt)

    def q(self, M):
        """Queries [B, Hq, M, D]."""
        B, Hkv, D = self.u.shape[0], self.u.shape[1], self.u.shape[3]
        G = self.c["Hq"] // Hkv
        x = self.src.normal(B, Hkv, G * M, D)
        if self.heavy:
            x += 2.0 * self.u
        return x.view(B, Hkv * G, M, D).to(DT[self.c["dtype"]])


def segment_names(c):
    """Segments of a cache in logical order (a protected tail comes last)."""
    return [s for s in ("keep", "kept", "pack") if c[s] > 0]


def cache_inputs(c, seed):
    """Raw rows of every segment (before quantisation) and what the steps add."""
    src = Source(seed)
    h = Heads(src, c, c.get("heavy"))
    x = {"rows": {s: h.kv(c[s], c.get("heavy") and s == "kept") for s in segment_names(c)}}
    if c["kind"] == "decode":
        x["tail"] = h.kv(c["tail"])
        x["new"] = [h.kv(c["M"]) for _ in range(c["steps"])]
        x["q"] = [h.q(c["M"]) for _ in range(c["steps"])]
    else:
        x["q"] = h.q(c["M"])
    return x


def batch_rows(c):
    """Kept rows and tail rows of every request."""
    R = c["R"]
    lo, hi = min(c["kept_min"], c["kept_max"]), max(c["kept_min"], c["kept_max"])
    return [(lo + (hi - lo) * r // max(1, R - 1), 1 + (r * c["tail"]) // R) for r in range(R)]


def batch_inputs(c, seed):
    src = Source(seed)
    h = Heads(src, c, 0)
    x = {"req": []}
    for r, (kept, tail) in enumerate(batch_rows(c)):
        parts = {"kept": h.kv(kept, b=r)}
        if c["pack"]:
            parts["pack"] = h.kv(c["pack"] - 3 * r if c["pack"] > 4 * c["R"] else c["pack"], b=r)
        parts["tail"] = h.kv(tail, b=r)
        x["req"].append(parts)
    x["q"] = h.q(c["M"])
    return x


def latent_bits(c):
    """Code width of each KV head of the latent: mostly int4."""
    return [2 if i % 4 == 3 else 4 for i in range(c["B"] * c["Hkv"])]


def denoise_inputs(c, seed):
    src = Source(seed)
    h = Heads(src, c, 0)
    return {"text": h.kv(c["text"]), "latent": h.kv(c["latent"]), "q": h.q(c["M"])}


def score_inputs(c, seed):
    src = Source(seed)
    h = Heads(src, c, c["heavy"])
    x = {"text": h.kv(c["text"]), "vit": h.kv(c["vit"], c["heavy"])}
    if c["pack"]:
        x["pack"] = h.kv(c["pack"])
    x["q"] = h.q(c["W"])
    return x


def compress_inputs(c, seed):
    src = Source(seed)
    h = Heads(src, c, 0)
    BH = c["B"] * c["Hkv"]
    # heavy-tailed probability sums, as a scoring pass leaves them
    s = torch.exp(1.5 * src.student(BH, c["rows"]).clamp_(-4, 6))
    s = s / s.sum(-1, keepdim=True) * (32 * c["Hq"] // c["Hkv"])
    return {"scores": s, "vit": h.kv(c["rows"]), "text": h.kv(c["quant"])}


def request_workload(c):
    """The repository's tiny workload at the case's sizes."""
    S = workloads.SegSpec
    return workloads.scaled(workloads.TINY_UNDERSTANDING, W=c["W"], segments=(
        S("text", c["text"], "keep", "f16"), S("vit", c["vit"], "evict", "f32", keep_ratio=c["ratio"]),
        S("vae", c["vae"], "quant", "f32", bits=c["bits"], group=c["group"])))


def request_inputs(c, seed):
    w, src = request_workload(c), Source(seed)
    B, Hq, Hkv, D = w.B, w.Hq, w.Hkv, w.D
    scale = torch.ones(B, Hkv, 1, D, device="cuda")
    scale[..., torch.randperm(D, generator=src.g, device="cuda")[:4]] = 10.0
    x = {"seg_k": [], "seg_v": []}
    for s in w.segments:
        x["seg_k"].append((src.normal(B, Hkv, s.n, D) * scale).to(DT[s.dtype]))
        x["seg_v"].append(src.normal(B, Hkv, s.n, D).to(DT[s.dtype]))
    x["q_obs"] = src.normal(B, Hq, w.W, D)
    x["q_dec"] = src.normal(1, B, Hq, 1, D)
    return w, x


# ---------------------------------------------------------------- states

def packed(shape, k, v, c, bits, capacity=0, head_bits=None):
    B, Hkv, n, D = k.shape
    seg = uc.packed_segment(B, Hkv, n, D, c["group"], k.dtype, bits=bits, head_bits=head_bits, capacity=capacity)
    uc.uc_quantize_segment(shape, k, v, n, seg)
    return seg


def workspace(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device="cuda")


def prepare(c, seed):
    s = {"case": c, "kind": c["kind"]}
    if c["kind"] == "request":
        w, x = request_inputs(c, seed)
        s.update(run=Run(w, x), o=torch.empty(w.B, w.Hq, 1, w.D, device="cuda"),
                 lse=torch.empty(w.B, w.Hq, 1, device="cuda"))
        return s
    B, Hq, Hkv, D = c.get("B", c.get("R")), c["Hq"], c["Hkv"], c["D"]
    shape = s["shape"] = uc.make_shape(B, Hq, Hkv, D)
    s["sm"] = scale_of(D)
    dt = uc.NAME_DT[c["dtype"]]

    def outputs(M, n=1):
        s["o"] = torch.empty(n, B, Hq, M, D, device="cuda")
        s["lse"] = torch.empty(n, B, Hq, M, device="cuda")

    if c["kind"] in ("decode", "prefill"):
        x = cache_inputs(c, seed)
        M, stream = c["M"], c.get("api") == "stream"
        segs = []
        for name in segment_names(c):
            k, v = x["rows"][name]
            if name == "pack":
                room = c["pack"] + c["steps"] * c["M"] if stream else 0
                segs.append(packed(shape, k, v, c, c["bits"], capacity=room))
            else:
                segs.append(uc.dense_segment(k, v))
        if c["kind"] == "decode":
            k, v = (torch.zeros(B, Hkv, c["capacity"], D, dtype=DT[c["dtype"]], device="cuda") for _ in range(2))
            k[:, :, :c["tail"]], v[:, :, :c["tail"]] = x["tail"]
            segs.append(uc.dense_segment(k, v, n_rows=c["capacity"]))
            s["at"] = len(segs) - (2 if stream else 1)  # the segment that grows
            if stream:
                segs[s["at"]].n_rows = c["pack"] + c["steps"] * c["M"]
            # enough for an execution plan as well
            s["ws"] = workspace(uc.uc_attend_workspace_size(shape, segs, dt, M))
            segs[-1].n_rows = c["tail"]
            if c["api"] == "plan":
                plan = uc.AttendPlan(shape, segs, s["at"], DT[c["dtype"]], M, s["sm"])
                s["ws"] = plan.ws
                plan.close()
            outputs(M, c["steps"])
        else:
            s["ws"] = workspace(uc.uc_attend_workspace_size(shape, segs, dt, M))
            outputs(M)
            s["seg_lse"] = torch.empty(B, Hq, M, len(segs), device="cuda")
        s.update(segs=segs, x={n: x[n] for n in x if n in ("q", "new")})
    elif c["kind"] == "batch":
        x = batch_inputs(c, seed)
        one = uc.make_shape(1, Hq, Hkv, D)
        s["reqs"] = []
        for parts in x["req"]:
            s["reqs"].append([packed(one, *parts[n], c, c["bits"]) if n == "pack" else uc.dense_segment(*parts[n])
                              for n in ("pack", "kept", "tail") if n in parts])
        s["ws"] = workspace(uc.uc_attend_batch_workspace_size(shape, s["reqs"], dt, c["M"]))
        s["q"] = x["q"]
        outputs(c["M"])
    elif c["kind"] == "denoise":
        x = denoise_inputs(c, seed)
        s["text"] = uc.dense_segment(*x["text"])
        s["latent"] = uc.packed_segment(B, Hkv, c["latent"], D, c["group"], DT[c["dtype"]], head_bits=latent_bits(c))
        s["rows"], s["q"] = x["latent"], x["q"]
        s["ws"] = workspace(uc.uc_attend_workspace_size(shape, [s["text"], s["latent"]], dt, c["M"]))
        outputs(c["M"])
        s["seg_lse"] = torch.empty(B, Hq, c["M"], 2, device="cuda")
        s["mass"] = torch.empty(B, Hkv, 2, device="cuda")
    elif c["kind"] == "score":
        x = score_inputs(c, seed)
        segs = [uc.dense_segment(*x["text"]), uc.dense_segment(*x["vit"])]
        if c["pack"]:
            segs.append(packed(shape, *x["pack"], c, c["bits"]))
        s.update(segs=segs, q=x["q"], ws=workspace(uc.uc_score_workspace_size(shape, segs, c["W"])),
                 scores=[torch.empty(B, Hkv, g.n_rows, device="cuda") for g in segs],
                 mass=torch.empty(B, Hkv, len(segs), device="cuda"))
        if c["columns"]:  # the attention pass whose row log-sum-exps the scores go by
            o = torch.empty(B, Hq, c["W"], D, device="cuda")
            s["row_lse"] = torch.empty(B, Hq, c["W"], device="cuda")
            uc.uc_attend_mixed(shape, segs, x["q"], c["W"], s["sm"], o, s["row_lse"])
    else:
        x = compress_inputs(c, seed)
        dst = [torch.empty(B * Hkv, c["k"], D, dtype=DT[c["dtype"]], device="cuda") for _ in range(2)]
        s.update(scores=x["scores"], src=[t.view(B * Hkv, c["rows"], D) for t in x["vit"]], dst=dst,
                 keep=torch.empty(B * Hkv, c["k"], dtype=torch.int32, device="cuda"), text=x["text"],
                 packed=uc.packed_segment(B, Hkv, c["quant"], D, c["group"], DT[c["dtype"]], bits=c["bits"]))
    return s


# ---------------------------------------------------------------- one pass

def run(s):
    c, kind = s["case"], s["kind"]
    if kind == "request":
        r = s["run"]
        r.compress()
        r.decode_step(0, s["o"], s["lse"])
        return {"o": s["o"], "lse": s["lse"], "scores": r.scores[1], "mass": r.mass, "kept": r.mixed[1].t["k"],
                "codes": r.mixed[2].t["codes_k"], "scale": r.mixed[2].t["scale_k"]}
    shape, sm = s["shape"], s["sm"]
    if kind == "decode":
        segs, at, M = s["segs"], s["at"], c["M"]
        q, new = s["x"]["q"], s["x"]["new"]
        segs[at].n_rows = c["pack"] if c["api"] == "stream" else c["tail"]  # the request starts again from here
        if c["api"] == "plan":
            plan = uc.AttendPlan(shape, segs, at, DT[c["dtype"]], M, sm, ws=s["ws"])
        for t in range(c["steps"]):
            k, v = new[t]
            if c["api"] == "plan":
                plan.attend_append(k, v, M, q[t], s["o"][t], s["lse"][t])
            elif c["api"] == "append":
                uc.uc_attend_append(shape, segs, at, k, v, M, q[t], M, sm, s["o"][t], s["lse"][t], ws=s["ws"])
            else:
                uc.uc_stream_append(shape, segs[at], k, v, M)
                uc.uc_attend_mixed(shape, segs, q[t], M, sm, s["o"][t], s["lse"][t], ws=s["ws"])
        if c["api"] == "plan":
            plan.close()
        t = segs[at].t
        if c["api"] == "stream":
            return {"o": s["o"], "lse": s["lse"], "codes": t["codes_k"], "scale": t["scale_k"], "min": t["min_v"]}
        return {"o": s["o"], "lse": s["lse"], "tail_k": t["k"], "tail_v": t["v"]}
    if kind == "prefill":
        uc.uc_attend_mixed(shape, s["segs"], s["x"]["q"], c["M"], sm, s["o"][0], s["lse"][0],
                           s["seg_lse"] if c["stats"] else None, ws=s["ws"])
        return {"o": s["o"], "lse": s["lse"], **({"seg_lse": s["seg_lse"]} if c["stats"] else {})}
    if kind == "batch":
        uc.uc_attend_batch(shape, s["reqs"], s["q"], c["M"], sm, s["o"][0], s["lse"][0], ws=s["ws"])
        return {"o": s["o"], "lse": s["lse"]}
    if kind == "denoise":
        uc.uc_quantize_segment(shape, *s["rows"], c["latent"], s["latent"])
        uc.uc_attend_mixed(shape, [s["text"], s["latent"]], s["q"], c["M"], sm, s["o"][0], s["lse"][0], s["seg_lse"],
                           ws=s["ws"])
        uc.uc_segment_mass(shape, c["M"], 2, s["lse"][0], s["seg_lse"], s["mass"])
        return {"o": s["o"], "lse": s["lse"], "seg_lse": s["seg_lse"], "mass": s["mass"],
                "codes": s["latent"].t["codes_k"], "scale": s["latent"].t["scale_k"]}
    if kind == "score":
        if c["columns"]:
            uc.uc_score_columns(shape, s["segs"], s["q"], c["W"], sm, s["row_lse"], c["W"], s["scores"], s["mass"],
                                ws=s["ws"])
        else:
            uc.uc_score_importance(shape, s["segs"], s["q"], c["W"], sm, s["scores"], s["mass"], ws=s["ws"])
        return {"scores": s["scores"], "mass": s["mass"]}
    uc.uc_select_keep(s["scores"], c["k"], c["recent"], s["keep"], *s["src"], *s["dst"])
    uc.uc_quantize_segment(shape, *s["text"], c["quant"], s["packed"])
    t = s["packed"].t
    return {"keep": s["keep"], "k": s["dst"][0], "v": s["dst"][1],
            **{n: t[n] for n in ("codes_k", "codes_v", "scale_k", "min_k", "scale_v", "min_v", "tail_k", "tail_v")}}


# ---------------------------------------------------------------- the work of a pass

def packed_bytes(n, D, G, bits, size):
    """Bytes of one head's packed segment of n rows: codes, scales and minima, unquantised remainder."""
    full = n // G * G
    return full * 2 * D * bits // 8 + 2 * 4 * (full // G * D + full * (D // G)) + (n - full) * 2 * D * size


def work(c):
    if c["kind"] == "request":
        D, Hq, kept = 64, 4, int(c["ratio"] * c["vit"])
        rows = c["text"] + c["vit"] + c["vae"]
        attended = c["text"] * 4 * D + kept * 8 * D + packed_bytes(c["vae"], D, c["group"], c["bits"], 4)
        # keys scored, rows kept and codes made, then the compressed cache read
        b = (c["text"] * 2 + (c["vit"] + c["vae"]) * 4) * D + 2 * kept * 8 * D + c["vae"] * 4 * D + 2 * attended
        return {"bytes": b, "flops": 2 * Hq * c["W"] * rows * D + 4 * Hq * D * (c["text"] + kept + c["vae"])}
    B, Hq, Hkv, D, e = c.get("B", c.get("R")), c["Hq"], c["Hkv"], c["D"], SIZE[c["dtype"]]
    if c["kind"] == "batch":
        b = f = 0
        for r, (kept, tail) in enumerate(batch_rows(c)):
            n = c["pack"] - 3 * r if c["pack"] > 4 * c["R"] else c["pack"]
            b += Hkv * ((kept + tail) * 2 * D * e + packed_bytes(n, D, c["group"], c["bits"], e))
            f += 4 * Hq * c["M"] * D * (kept + tail + n)
        return {"bytes": b + B * Hq * c["M"] * (D * (e + 4) + 4), "flops": f}
    if c["kind"] in ("decode", "prefill"):
        steps, M = c.get("steps", 1), c["M"]
        dense = c["keep"] + c["kept"] + c.get("tail", 0)
        rows = dense + c["pack"]
        kv = dense * 2 * D * e + packed_bytes(c["pack"], D, c["group"], c["bits"], e)
        # each step reads the cache and the rows added so far, and stores its own
        grow = M * 2 * D * e * (steps * (steps + 1) // 2 + steps) if c["kind"] == "decode" else 0
        io = steps * B * Hq * M * (D * (e + 4) + 4)
        return {"bytes": B * Hkv * (steps * kv + grow) + io, "flops": 4 * B * Hq * M * D * rows * steps}
    if c["kind"] == "denoise":
        n, bits = c["latent"], latent_bits(c)
        codes = sum(packed_bytes(n, D, c["group"], b, e) for b in bits)
        rows = B * Hkv * (n + c["text"]) * 2 * D * e
        return {"bytes": rows + 2 * codes + B * Hq * c["M"] * (D * (e + 4) + 4 * 3),
                "flops": 4 * B * Hq * c["M"] * D * (n + c["text"])}
    if c["kind"] == "score":
        rows = c["text"] + c["vit"]
        keys = rows * D * e + packed_bytes(c["pack"], D, c["group"], c["bits"], e) // 2
        return {"bytes": B * Hkv * (keys + (rows + c["pack"]) * 4) + B * Hq * c["W"] * D * e,
                "flops": 2 * B * Hq * c["W"] * D * (rows + c["pack"])}
    n = c["quant"]
    return {"bytes": B * Hkv * (c["rows"] * 4 + c["k"] * (4 + 2 * 2 * D * e) + n * 2 * D * e +
                                packed_bytes(n, D, c["group"], c["bits"], e)), "flops": 0}


def tolerance(c):
    # measured against exact(), times about four
    if c["kind"] == "compress":
        return "exact"  # selected rows, codes, scales and minima are defined bit for bit
    if c["kind"] == "request":
        return {"rel": 4e-6, "differ": 0.01}  # 32 bits throughout: 8e-7 seen; a tie at the cut may fall either way
    if c["kind"] == "score":
        return {"rel": 4e-6}  # 32-bit exponentials, sums kept wider: 8e-7 seen
    if c["kind"] in ("prefill", "denoise") and c["dtype"] == "bf16" and c["D"] == 128:
        return {"rel": 8e-4}  # probabilities with 11 bits of mantissa: 2e-4 seen
    return {"rel": 1e-5}  # probabilities with 16 bits or more: 2.3e-6 seen


# ---------------------------------------------------------------- 64 bits

def quantised(k, v, G, bits):
    """(K, V) in 64 bits as a packed segment of these rows stands for them, and
    the codes' scales and minima.  bits: one width, or one per (b, h)."""
    B, H, n, D = k.shape
    full = n // G * G
    if isinstance(bits, int):
        bits = [bits] * (B * H)
    qmax = torch.tensor([2.0 ** b - 1 for b in bits], device="cuda").view(B, H, 1, 1, 1)
    out, meta = [], []
    for x, shape, axis in ((k, (B, H, full // G, G, D), 3), (v, (B, H, full, D // G, G), 4)):
        y = x[:, :, :full].float().reshape(shape)
        mn, mx = y.amin(axis, keepdim=True), y.amax(axis, keepdim=True)
        s = ((mx - mn).double() / qmax.double()).float()
        # the definition is in 32 bits: the quotient is rounded to 32 before it is rounded to a code
        code = ((y - mn).double() / s.double()).float().round_()
        code = torch.where(s > 0, code.clamp_(min=0).minimum(qmax), torch.zeros_like(code))
        z = (code.double() * s.double() + mn.double()).float().to(x.dtype)
        out.append(torch.cat([z.reshape(B, H, full, D), x[:, :, full:]], 2).double())
        meta += [s.squeeze(axis), mn.squeeze(axis)]
        del y, code, z
    return out[0], out[1], meta


def attend64(segs, q, D):
    """softmax(q K^T / sqrt(D)) V over segments [(K, V)] of one request batch:
    o, lse and per-segment lse in 64 bits, a KV head at a time."""
    B, Hq, M, _ = q.shape
    Hkv = segs[0][0].shape[1]
    G = Hq // Hkv
    o = torch.empty(B, Hq, M, D, dtype=torch.float64, device="cuda")
    lse = torch.empty(B, Hq, M, dtype=torch.float64, device="cuda")
    per = torch.empty(B, Hq, M, len(segs), dtype=torch.float64, device="cuda")
    for b in range(B):
        for h in range(Hkv):
            heads = slice(h * G, (h + 1) * G)
            x = q[b, heads].double().reshape(G * M, D) * scale_of(D)
            s = [x @ k[b, h].double().t() for k, _ in segs]
            each = torch.stack([t.logsumexp(-1) for t in s], -1)
            total = each.logsumexp(-1)
            acc = sum(torch.exp(t - total[:, None]) @ v[b, h].double() for t, (_, v) in zip(s, segs))
            o[b, heads], lse[b, heads] = acc.view(G, M, D), total.view(G, M)
            per[b, heads] = each.view(G, M, -1)
            del s
    return o, lse, per


def score64(keys, q, D, lse=None):
    """Probability that each key of each segment gets, summed over the rows of
    q [B, Hq, W, D] of its KV head, and the segments' masses."""
    B, Hq, W, _ = q.shape
    Hkv = keys[0].shape[1]
    G = Hq // Hkv
    out = [torch.empty(B, Hkv, k.shape[2], dtype=torch.float64, device="cuda") for k in keys]
    for b in range(B):
        for h in range(Hkv):
            x = q[b, h * G:(h + 1) * G].double().reshape(G * W, D) * scale_of(D)
            s = torch.cat([x @ k[b, h].double().t() for k in keys], -1)
            p = torch.softmax(s, -1).sum(0)
            for t, part in zip(out, p.split([k.shape[2] for k in keys])):
                t[b, h] = part
    return out, torch.stack([t.sum(-1) for t in out], -1)


def exact(c, seed):
    kind, D = c["kind"], c.get("D", 64)
    if kind == "request":
        w, x = request_inputs(c, seed)
        k, v = x["seg_k"], x["seg_v"]
        scores, mass = score64(k, x["q_obs"], D)
        n_kept = int(math.floor(c["ratio"] * c["vit"]))
        order = scores[1].argsort(dim=-1, descending=True, stable=True)[..., :n_kept].sort(-1).values
        at = order[..., None].expand(-1, -1, -1, D)
        kept = k[1].gather(2, at), v[1].gather(2, at)
        pk, pv, meta = quantised(k[2], v[2], c["group"], c["bits"])
        o, lse, _ = attend64([(k[0], v[0]), kept, (pk, pv)], x["q_dec"][0], D)
        return {"o": o, "lse": lse, "scores": scores[1], "mass": mass, "kept": None, "codes": None, "scale": meta[0]}
    if kind in ("decode", "prefill"):
        x = cache_inputs(c, seed)
        stream, segs = c.get("api") == "stream", []
        for n in segment_names(c):
            segs.append(quantised(*x["rows"][n], c["group"], c["bits"])[:2] if n == "pack" else x["rows"][n])
        if kind == "prefill":
            o, lse, per = attend64(segs, x["q"], D)
            return {"o": o[None], "lse": lse[None], **({"seg_lse": per} if c["stats"] else {})}
        os, ls = [], []
        tail = x["tail"]
        rows = x["rows"].get("pack")
        for t in range(c["steps"]):
            if stream:
                rows = tuple(torch.cat([a, b], 2) for a, b in zip(rows, x["new"][t]))
                segs[-1] = quantised(*rows, c["group"], c["bits"])[:2]
            else:
                tail = tuple(torch.cat([a, b], 2) for a, b in zip(tail, x["new"][t]))
            o, lse, _ = attend64(segs + [tail], x["q"][t], D)
            os.append(o)
            ls.append(lse)
        out = {"o": torch.stack(os), "lse": torch.stack(ls)}
        if stream:
            return {**out, "codes": None, "scale": None, "min": None}
        pad = c["capacity"] - tail[0].shape[2]
        return {**out, **{n: torch.nn.functional.pad(t.double(), (0, 0, 0, pad)) for n, t in zip(("tail_k", "tail_v"), tail)}}
    if kind == "batch":
        x = batch_inputs(c, seed)
        os, ls = [], []
        for r, parts in enumerate(x["req"]):
            segs = [quantised(*parts[n], c["group"], c["bits"])[:2] if n == "pack" else parts[n] for n in parts]
            o, lse, _ = attend64(segs, x["q"][r:r + 1], D)
            os.append(o)
            ls.append(lse)
        return {"o": torch.cat(os)[None], "lse": torch.cat(ls)[None]}
    if kind == "denoise":
        x = denoise_inputs(c, seed)
        k, v, meta = quantised(*x["latent"], c["group"], latent_bits(c))
        o, lse, per = attend64([x["text"], (k, v)], x["q"], D)
        G = c["Hq"] // c["Hkv"]
        mass = torch.exp(per - lse[..., None]).view(c["B"], c["Hkv"], G * c["M"], 2).sum(2)
        return {"o": o[None], "lse": lse[None], "seg_lse": per, "mass": mass, "codes": None, "scale": meta[0]}
    if kind == "score":
        x = score_inputs(c, seed)
        keys = [x["text"][0], x["vit"][0]]
        if c["pack"]:
            keys.append(quantised(*x["pack"], c["group"], c["bits"])[0])
        scores, mass = score64(keys, x["q"], D)
        return {"scores": scores, "mass": mass}
    x = compress_inputs(c, seed)
    n = c["rows"] - c["recent"]
    s = x["scores"][:, :n]
    keep = s.argsort(dim=-1, descending=True, stable=True)[:, :c["k"] - c["recent"]].sort(-1).values
    last = torch.arange(n, c["rows"], device="cuda").expand(s.shape[0], -1)
    at = torch.cat([keep, last], 1).view(c["B"], c["Hkv"], -1, 1).expand(-1, -1, -1, D)
    rows = [t.gather(2, at).view(s.shape[0], -1, D) for t in x["vit"]]
    _, _, meta = quantised(*x["text"], c["group"], c["bits"])
    full = c["quant"] // c["group"] * c["group"]
    tail = [t[:, :, full:] for t in x["text"]]
    return {"keep": None, "k": rows[0], "v": rows[1], "codes_k": None, "codes_v": None, "scale_k": meta[0],
            "min_k": meta[1], "scale_v": meta[2], "min_v": meta[3], "tail_k": tail[0], "tail_v": tail[1]}
