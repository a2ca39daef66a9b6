"""The work that users of this framework have it do, as cases that can be timed.

A case names a model (one of the five configurations of ``synth``), the call or calls a camera
pipeline makes, the number and size of its cameras, the frames' element type and how much of
every frame is critical.  Frames, boxes and random weights are drawn on the GPU from the seed;
a state holds what a serving program keeps: the context with its weights and its output buffers.

The paper-side calls of a pipeline:
  multilevel  coarse stage, selection and fine stage of a batch in one call
  coarse      the coarse subtask alone, as a scheduler issues it
  fine        the fine subtask alone: selection, then the mixed encode with the cached tokens
  stages      coarse encode, decode, region proposal, selection of the hard frames, fine encode:
              the two subtasks of a detector with nothing of the host between them
  decode      object queries of a batch from its encoded tokens
  select      the integer selection alone
"""
import math
import random

import numpy as np
import torch

from paper_2505_23317_amd import cfdetr, synth

N_QUERIES = 300     # object queries of a frame, and decoder layers behind them
DEC_LAYERS = 6


def _case(name, call, model, cameras, height, width, frames="bf16", lo=0.0, hi=0.0, objects=0):
    c = {"call": call, "model": model, "cameras": cameras, "height": height, "width": width,
         "frames": frames, "critical_lo": lo, "critical_hi": hi, "objects": objects}
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest call: which cells to refine, for six cameras; launches and host time.
        _case("select_six", "select", 3, 6, 640, 640, lo=0.0, hi=0.5),
        # A tiny model on one small fp32 frame: latency of the whole chain of launches.
        _case("tiny_frame_f32", "multilevel", 1, 1, 128, 128, "f32", lo=0.1, hi=0.3),
        # One camera of a vehicle, about a quarter of the area critical.
        _case("one_camera", "multilevel", 2, 1, 640, 640, lo=0.25, hi=0.25),
        # The surround view: six cameras, every one with its own critical share.
        _case("six_cameras", "multilevel", 3, 6, 640, 640, lo=0.0, hi=0.5),
        # A coarse subtask on its own: one wide fp32 frame, an odd number of token rows.
        _case("coarse_wide_f32", "coarse", 4, 1, 736, 1280, "f32"),
        # A fine subtask on its own: one high-resolution frame whose coarse stage has run.
        _case("fine_one_camera", "fine", 4, 1, 1280, 1280, lo=0.4, hi=0.4),
        # Four high-resolution cameras, from nothing critical to everything.
        _case("high_res", "multilevel", 4, 4, 1280, 1280, lo=0.0, hi=1.0),
        # The worst case a scheduler has to plan for: eight frames, everything critical.
        _case("high_res_all", "multilevel", 4, 8, 1280, 1280, lo=1.0, hi=1.0),
        # Three granularities, twelve cameras, boxes of mixed criticality.
        _case("three_level", "multilevel", 5, 12, 1024, 1024, objects=12),
        # The same model on three small frames: few tokens for a wide model.
        _case("three_level_small", "multilevel", 5, 3, 576, 960, objects=5),
        # Object queries of four cameras from their coarse tokens.
        _case("decode_coarse", "decode", 4, 4, 1280, 1280),
        # The detector's two stages on six cameras, two of them easy, queries after the first.
        _case("two_stages", "stages", 3, 6, 640, 640),
    ]


# frame sides and camera counts a model is used with
_RANGES = {1: (64, 256, 8), 2: (256, 960, 2), 3: (256, 960, 12), 4: (512, 1280, 8), 5: (512, 1280, 12)}


def draw(rng: random.Random):
    def log_uniform(a, b):
        return math.exp(rng.uniform(math.log(a), math.log(b)))

    call = rng.choice(["multilevel"] * 7 + ["coarse", "fine", "stages", "decode", "select"])
    model = rng.choice([1, 2, 3, 4, 4, 5, 5] if call != "stages" else [2, 3, 4])
    p0 = synth.config(model).patch[0]
    side_lo, side_hi, cams = _RANGES[model]
    height, width = (p0 * max(1, round(log_uniform(side_lo, side_hi) / p0)) for _ in range(2))
    cameras = max(1, min(cams, round(log_uniform(0.7, cams + 0.4))))
    lo, hi = sorted(round(rng.uniform(0.0, 1.0), 3) for _ in range(2))
    tiered = model == 5
    c = _case(None, call, model, cameras, height, width,
              "f32" if model == 1 or rng.random() < 0.2 else "bf16",
              0.0 if tiered else lo, 0.0 if tiered else hi, rng.randint(3, 16) if tiered else 0)
    most = work(listed()[7])["flops"]
    while c["cameras"] > 1 and work(c)["flops"] > most:
        c["cameras"] -= 1
    return c


# ---- inputs ------------------------------------------------------------------------
def _config(case):
    return synth.replace(synth.config(case["model"]), B=case["cameras"], H=case["height"],
                         W=case["width"], image_dtype=case["frames"])


def _rand_box(rng, cfg):
    """A box with sides of the model's side law, as a half-open pixel rectangle."""
    hi = min(cfg.side_hi, cfg.H, cfg.W)
    lo = min(cfg.side_lo, hi)
    if cfg.box_rule == "single48":
        lo, hi = 16, 64
    w, h = (int(v) for v in rng.integers(lo, hi + 1, 2))
    x, y = int(rng.integers(0, cfg.W - w + 1)), int(rng.integers(0, cfg.H - h + 1))
    return x, y, x + w, y + h


def _boxes(cfg, case, seed):
    """Boxes of a batch: per frame [(box, tier)].  Either a number of objects of mixed tiers, or
    random boxes until their union covers the frame's critical share of the coarse cells (the
    shares are spread evenly over the case's range and dealt out to the frames)."""
    rng = np.random.default_rng(seed)
    top, p0 = cfg.n_levels - 1, cfg.patch[0]
    rows, cols = cfg.grid(0)
    out = []
    if case["objects"]:
        for f in range(cfg.B):
            n = max(1, int(rng.poisson(case["objects"])))
            u = rng.uniform(0.0, 1.0, n)
            out.append([(_rand_box(rng, cfg), top if x < 0.3 else max(top - 1, 0) if x < 0.7 else 0)
                        for x in u])
        return out
    span = case["critical_hi"] - case["critical_lo"]
    shares = [case["critical_lo"] + span * (f + 0.5) / cfg.B for f in range(cfg.B)]
    for share in rng.permutation(shares):
        if share >= 1.0:
            out.append([((0, 0, cfg.W, cfg.H), top)])
            continue
        hit, frame = np.zeros((rows, cols), dtype=bool), []
        while hit.sum() < share * rows * cols and len(frame) < 2000:
            b = _rand_box(rng, cfg)
            hit[b[1] // p0:-(-b[3] // p0), b[0] // p0:-(-b[2] // p0)] = True
            frame.append((b, top))
        out.append(frame)
    return out


def _tokens(cfg, frames):
    """Tokens of every frame at every level [B][levels] for the given boxes."""
    counts = []
    for frame in frames:
        alive = np.ones(cfg.grid(0), dtype=bool)
        row = []
        for level in range(cfg.n_levels):
            p = cfg.patch[level]
            split = np.zeros(cfg.grid(level), dtype=bool)
            if level + 1 < cfg.n_levels:
                for (x0, y0, x1, y1), tier in frame:
                    if tier > level:
                        split[y0 // p:-(-y1 // p), x0 // p:-(-x1 // p)] = True
            row.append(int((alive & ~split).sum()))
            alive = np.kron(alive & split, np.ones((2, 2), dtype=bool)).astype(bool)
        counts.append(row)
    return counts


class _Draw:
    """Random device tensors from one seed."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)

    def normal(self, shape, std=1.0, mean=0.0, dtype=torch.float32):
        x = torch.randn(shape, generator=self.gen, device="cuda")
        return x.mul_(std).add_(mean).to(dtype)

    def uniform(self, shape):
        return torch.rand(shape, generator=self.gen, device="cuda")


def _frames(cfg, frames, seed):
    """Gaussian-noise frames with rectangles of constant colour painted on."""
    rnd = _Draw(seed)
    img = rnd.normal((cfg.B, 3, cfg.H, cfg.W), 0.25, 0.5).clamp_(0.0, 1.0)
    colours = rnd.uniform((cfg.B, 20, 3, 1, 1))
    rng = np.random.default_rng(seed)
    for f in range(cfg.B):
        known = [b for b, _ in frames[f][:12]] if frames else []
        for k in range(20):
            x0, y0, x1, y1 = known[k] if k < len(known) else _rand_box(rng, cfg)
            if (x1 - x0) * (y1 - y0) < cfg.H * cfg.W // 2:
                img[f, :, y0:y1, x0:x1] = colours[f, k]
    return img.to(torch.bfloat16) if cfg.image_dtype == "bf16" else img


def _encoder_weights(cfg, seed):
    rnd, d, F, L = _Draw(seed), cfg.d, cfg.ffn, cfg.layers
    bf = torch.bfloat16
    w = {}
    for level, p in enumerate(cfg.patch):
        w[f"w_embed{level}"] = rnd.normal((d, 3 * p * p), 0.02, dtype=bf)
        w[f"b_embed{level}"] = rnd.normal((d,), 0.02)
    for name, shape in (("w_qkv", (L, 3 * d, d)), ("w_o", (L, d, d)), ("w_ff1", (L, F, d)),
                        ("w_ff2", (L, d, F))):
        w[name] = rnd.normal(shape, 0.02, dtype=bf)
    for name, shape in (("b_qkv", (L, 3 * d)), ("b_o", (L, d)), ("b_ff1", (L, F)), ("b_ff2", (L, d)),
                        ("ln1_b", (L, d)), ("ln2_b", (L, d)), ("lnf_b", (d,))):
        w[name] = rnd.normal(shape, 0.02)
    for name, shape in (("ln1_g", (L, d)), ("ln2_g", (L, d)), ("lnf_g", (d,))):
        w[name] = rnd.normal(shape, 0.02, 1.0)
    return w


def _decoder_weights(cfg, seed):
    """Same law; query vectors and heads wider, so that boxes and confidences spread over (0, 1)."""
    rnd, d, F, L = _Draw(seed), cfg.d, cfg.ffn, DEC_LAYERS
    bf = torch.bfloat16
    w = {"query_embed": rnd.normal((N_QUERIES, d))}
    for name, shape, std in (("w_qkv", (L, 3 * d, d), 0.02), ("w_o", (L, d, d), 0.02),
                             ("w_q", (L, d, d), 0.02), ("w_kv", (L, 2 * d, d), 0.02),
                             ("w_o2", (L, d, d), 0.02), ("w_ff1", (L, F, d), 0.02),
                             ("w_ff2", (L, d, F), 0.02), ("w_cls", (1, d), 0.1),
                             ("w_box1", (d, d), 0.1), ("w_box2", (d, d), 0.1),
                             ("w_box3", (4, d), 0.1)):
        w[name] = rnd.normal(shape, std, dtype=bf)
    for name, shape in (("b_qkv", (L, 3 * d)), ("b_o", (L, d)), ("b_q", (L, d)), ("b_kv", (L, 2 * d)),
                        ("b_o2", (L, d)), ("b_ff1", (L, F)), ("b_ff2", (L, d)), ("ln1_b", (L, d)),
                        ("ln2_b", (L, d)), ("ln3_b", (L, d)), ("lnf_b", (d,)), ("b_cls", (1,)),
                        ("b_box1", (d,)), ("b_box2", (d,)), ("b_box3", (4,))):
        w[name] = rnd.normal(shape, 0.02)
    for name, shape in (("ln1_g", (L, d)), ("ln2_g", (L, d)), ("ln3_g", (L, d)), ("lnf_g", (d,))):
        w[name] = rnd.normal(shape, 0.02, 1.0)
    return w


class _DeviceEncoder(cfdetr.Encoder):
    """The binding's Encoder for weights that are on the device already."""

    def __init__(self, cfg, weights):
        self.cfg, self.act_bf16, self.dev = cfg, True, weights
        self.max_batch = cfg.B
        self.max_tokens = cfg.B * cfg.n_cells(cfg.n_levels - 1)
        self.n0 = cfg.n_cells(0)
        c, w = cfdetr.CfdetrConfig(), cfdetr.CfdetrWeights()
        c.n_levels = cfg.n_levels
        for level, p in enumerate(cfg.patch):
            c.patch[level] = p
            w.w_embed[level] = weights[f"w_embed{level}"].data_ptr()
            w.b_embed[level] = weights[f"b_embed{level}"].data_ptr()
        c.img_h, c.img_w = cfg.H, cfg.W
        c.d_model, c.n_heads, c.n_layers, c.d_ffn = cfg.d, cfg.heads, cfg.layers, cfg.ffn
        c.max_batch, c.max_tokens_total = self.max_batch, self.max_tokens
        c.image_dtype = cfdetr.CFDETR_BF16 if cfg.image_dtype == "bf16" else cfdetr.CFDETR_FP32
        c.act_dtype, c.ln_eps = cfdetr.CFDETR_BF16, 1e-5
        for name in ("ln1_g", "ln1_b", "w_qkv", "b_qkv", "w_o", "b_o", "ln2_g", "ln2_b", "w_ff1",
                     "b_ff1", "w_ff2", "b_ff2", "lnf_g", "lnf_b"):
            setattr(w, name, weights[name].data_ptr())
        self.c_cfg, self.c_w = c, w
        torch.cuda.synchronize()    # the weights are read on the library's own stream
        self.ctx = cfdetr.cfdetr_create(c, w)

    def attach_decoder(self, weights):
        self.dec_dev = weights
        w = cfdetr.CfdetrDecoderWeights()
        w.n_queries, w.n_layers = N_QUERIES, DEC_LAYERS
        for name in cfdetr.DECODER_FIELDS:
            setattr(w, name, weights[name].data_ptr())
        self.n_queries, self.c_dec = N_QUERIES, w
        torch.cuda.synchronize()
        cfdetr.cfdetr_decoder_attach(self.ctx, w)


def prepare(case, seed):
    cfg = _config(case)
    call, B = case["call"], cfg.B
    frames = _boxes(cfg, case, seed)
    s = {"call": call, "B": B}
    enc = s["enc"] = _DeviceEncoder(cfg, _encoder_weights(cfg, seed + 1))
    out = s["out"] = enc.alloc_outputs(B)
    flat = [e for frame in frames for e in frame]
    s["boxes"] = enc.upload_boxes([b for b, _ in flat], [t for _, t in flat],
                                  np.cumsum([0] + [len(frame) for frame in frames]))
    if call != "select":
        s["img"] = _frames(cfg, frames, seed + 2)
    if call in ("decode", "stages"):
        enc.attach_decoder(_decoder_weights(cfg, seed + 3))
        s["cu0"] = torch.arange(B + 1, dtype=torch.int32, device="cuda") * enc.n0
        s["coarse_q"] = torch.empty((B, N_QUERIES, 5), dtype=torch.float32, device="cuda")
    if call == "stages":
        # Regions come from the queries a tracker carries over from the frame before; one frame
        # in three is easy.
        q = synth.make_queries(cfg, seed, n_queries=N_QUERIES, easy_frames=tuple(range(2, B, 3)))
        s["tracked"] = torch.from_numpy(q).cuda()
        s["params"] = cfdetr.CfdetrRoiParams(0.8, 0.05, 1.0, 0.0, cfg.n_levels - 1)
        n = B * N_QUERIES
        s["roi"] = [torch.zeros((n, 4), dtype=torch.int32, device="cuda"),
                    torch.zeros(n, dtype=torch.uint8, device="cuda"),
                    torch.zeros(B + 1, dtype=torch.int32, device="cuda"),
                    torch.zeros(B, dtype=torch.int32, device="cuda"),
                    torch.zeros(B, dtype=torch.float32, device="cuda")]
    if call in ("fine", "decode"):
        enc.coarse_encode(s["img"], B, out["x0_cache"], out["y_coarse"])
    if call == "decode":
        s["memory"] = out["y_coarse"]
    torch.cuda.synchronize()
    return s


def run(s):
    enc, out, B, call = s["enc"], s["out"], s["B"], s["call"]
    boxes, tier, offs = s["boxes"]
    if call == "select":
        enc.select_fine(boxes, tier, offs, B, out["tok_desc"], out["cu_seqlens"], out["level_counts"])
        return {k: out[k] for k in ("tok_desc", "cu_seqlens", "level_counts")}
    if call == "multilevel":
        enc.multilevel_batch(s["img"], B, boxes, tier, offs, out)
        return {k: out[k] for k in ("y_coarse", "y_mixed", "tok_desc", "cu_seqlens", "level_counts")}
    if call == "coarse":
        enc.coarse_encode(s["img"], B, out["x0_cache"], out["y_coarse"])
        return {k: out[k] for k in ("x0_cache", "y_coarse")}
    if call == "fine":
        enc.select_fine(boxes, tier, offs, B, out["tok_desc"], out["cu_seqlens"], out["level_counts"])
        enc.fine_encode(s["img"], B, out["tok_desc"], out["cu_seqlens"], out["x0_cache"], out["y_mixed"])
        return {k: out[k] for k in ("y_mixed", "tok_desc", "cu_seqlens", "level_counts")}
    if call == "decode":
        enc.decode(s["memory"], s["cu0"], B, s["coarse_q"])
        return {"queries": s["coarse_q"]}
    # stages
    enc.coarse_encode(s["img"], B, out["x0_cache"], out["y_coarse"])
    enc.decode(out["y_coarse"], s["cu0"], B, s["coarse_q"])
    rb, rt, ro, hard, mean = s["roi"]
    enc.propose_rois(s["tracked"], s["params"], rb, rt, ro, hard, mean)
    enc.select_fine_hard(rb, rt, ro, hard, B, out["tok_desc"], out["cu_seqlens"], out["level_counts"])
    enc.fine_encode(s["img"], B, out["tok_desc"], out["cu_seqlens"], out["x0_cache"], out["y_mixed"])
    return {"y_coarse": out["y_coarse"], "y_mixed": out["y_mixed"], "coarse_q": s["coarse_q"],
            "tok_desc": out["tok_desc"], "cu_seqlens": out["cu_seqlens"], "hard": hard}


# ---- what a pass cannot do without ---------------------------------------------------
def _encode_flops(cfg, seqs):
    d, F, L = cfg.d, cfg.ffn, cfg.layers
    n, sq = sum(seqs), sum(t * t for t in seqs)
    return L * (n * (8.0 * d * d + 4.0 * d * F) + 4.0 * sq * d)


def _encode_weight_bytes(cfg):
    d, F, L = cfg.d, cfg.ffn, cfg.layers
    return L * (8.0 * d * d + 4.0 * d * F) + sum(6.0 * p * p * d for p in cfg.patch)


def _embed_flops(cfg, counts):
    return sum(6.0 * cfg.patch[level] ** 2 * cfg.d * n for level, n in enumerate(counts))


def _decode_work(cfg, seqs):
    d, F, L, Q = cfg.d, cfg.ffn, DEC_LAYERS, N_QUERIES
    n, rows = sum(seqs), len(seqs) * Q
    flops = L * (4.0 * n * d * d + rows * (12.0 * d * d + 4.0 * d * F)
                 + 4.0 * d * (len(seqs) * Q * Q + Q * n)) + rows * 4.0 * d * d
    return flops, 4.0 * n * d + L * 2.0 * (8.0 * d * d + 2.0 * d * F) + rows * 20.0


def work(case):
    cfg = _config(case)
    call, B, n0, d = case["call"], cfg.B, cfg.n_cells(0), cfg.d
    coarse, top = [n0] * B, cfg.n_levels - 1
    if call == "stages":
        frames = []
        for f, q in enumerate(synth.make_queries(cfg, 0, N_QUERIES, tuple(range(2, B, 3)))):
            mid = q[(q[:, 4] > 0.05) & (q[:, 4] <= 0.8)]
            lo, hi = mid[:, :2] - mid[:, 2:4] / 2, mid[:, :2] + mid[:, 2:4] / 2
            size = np.array([cfg.W, cfg.H])
            lo = np.clip(np.floor(lo * size), 0, size).astype(int)
            hi = np.clip(np.ceil(hi * size), 0, size).astype(int)
            frames.append([((a[0], a[1], b[0], b[1]), top) for a, b in zip(lo, hi)])
        counts = [c for f, c in enumerate(_tokens(cfg, frames)) if f % 3 != 2]
    else:
        frames = _boxes(cfg, case, 0)
        counts = _tokens(cfg, frames)
    mixed = [sum(c) for c in counts]
    by_level = [sum(c[level] for c in counts) for level in range(cfg.n_levels)]
    pixels = 3.0 * cfg.H * cfg.W * B * (2 if cfg.image_dtype == "bf16" else 4)
    fine_pixels = sum(n * 3.0 * p * p for n, p in zip(by_level[1:], cfg.patch[1:])) * (
        2 if cfg.image_dtype == "bf16" else 4)
    if call == "select":
        n = sum(len(frame) for frame in frames)
        cells = sum(cfg.n_cells(level) for level in range(top)) * B
        return {"bytes": 17.0 * n + 4.0 * sum(mixed) + 4.0 * B * (2 + cfg.n_levels), "flops": 4.0 * cells}
    if call == "decode":
        flops, nbytes = _decode_work(cfg, coarse)
        return {"bytes": nbytes, "flops": flops}
    flops, nbytes = 0.0, _encode_weight_bytes(cfg)
    if call in ("multilevel", "coarse", "stages"):
        flops += _embed_flops(cfg, [sum(coarse)]) + _encode_flops(cfg, coarse)
        nbytes += pixels + 4.0 * d * sum(coarse) * (1 if call == "multilevel" else 2)
    if call in ("multilevel", "fine", "stages"):
        flops += _embed_flops(cfg, [0] + by_level[1:]) + _encode_flops(cfg, mixed)
        nbytes += 4.0 * (d + 1) * sum(mixed)
        if call != "multilevel":    # the coarse stage's tokens, and the critical pixels once more
            nbytes += fine_pixels + 4.0 * d * by_level[0]
    if call == "stages":
        f, b = _decode_work(cfg, coarse)
        flops, nbytes = flops + f, nbytes + b
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Selections are integer work.  The encoder and decoder contract bf16 operands with fp32 sums:
    their results carry a few thousandths of the result's norm after twelve layers."""
    return "exact" if case["call"] == "select" else {"rel": 1e-2, "max": 0.1}
