"""The work that a user of this framework has it do, as measurable cases.

Every case is one pass through the public entry points of
``paper_2601_10819_amd.ops``: a forward alone (serving), a forward with the
backward through autograd (training), a frame of the FP8 form (quantise and
sample), the outside-in step (projection, sampling of the visible views,
backward) and the batch of uneven scenes. The sizes are those of the
workloads of ``synth.py`` and of ragged scenes between them; inputs are drawn on
the device by the same recipe (features N(0, 1), locations a little beyond
the image, weights a softmax over an anchor's samples).

``exact`` evaluates the same pass in float64 with plain torch.
"""
import math

import torch

from paper_2601_10819_amd import ops, synth

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
STRIDES = (4, 8, 16, 32)


def _case(name, kind, dtype, cams, img_h, img_w, anchors, batch=1, levels=4, channels=256,
          groups=8, points=13, out_of_view=0.0, logits=False, scenes=1, mixed=False):
    c = dict(kind=kind, dtype=dtype, batch=batch, cams=cams, img_h=img_h, img_w=img_w,
             levels=levels, channels=channels, groups=groups, anchors=anchors, points=points,
             out_of_view=out_of_view, logits=logits, scenes=scenes, mixed=mixed)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: a two-camera unit's forward, where launches and host work count
        _case("tiny_fwd_f32", "forward", "f32", 2, 128, 224, 128, channels=64, groups=4),
        # the same unit in training: the smallest step through autograd
        _case("tiny_step_f32", "train", "f32", 2, 128, 224, 128, channels=64, groups=4),
        # a six-camera rig at inference, one frame in BF16
        _case("rig6_fwd_bf16", "forward", "bf16", 6, 256, 704, 900),
        # the same rig in FP32 training
        _case("rig6_step_f32", "train", "f32", 6, 256, 704, 900),
        # a ragged site: odd image sizes that differ by camera, three levels, few keypoints,
        # 128 channels, FP16 storage, weights from the network's logits
        _case("ragged5_step_f16", "train", "f16", 5, 270, 492, 331, levels=3, channels=128,
              groups=4, points=7, logits=True, mixed=True),
        # the training configuration: two samples of 16 cameras, BF16, a quarter of the
        # keypoints out of each camera's view
        _case("train16_step_bf16", "train", "bf16", 16, 384, 640, 1800, batch=2,
              out_of_view=0.25),
        # the 64-camera scene at inference in the three storage types; FP8 codes are
        # made anew from each frame's features
        _case("scene64_fwd_f32", "forward", "f32", 64, 256, 448, 900),
        _case("scene64_fwd_bf16", "forward", "bf16", 64, 256, 448, 900),
        _case("scene64_frame_fp8", "frame_fp8", "f32", 64, 256, 448, 900),
        # the 64-camera scene in training
        _case("scene64_step_bf16", "train", "bf16", 64, 256, 448, 900),
        # the outside-in network: keypoints projected, visible views fused by their
        # scores, weights from logits, forward and backward
        _case("outside64_step_bf16", "fused", "bf16", 64, 256, 448, 900, logits=True),
        # twelve uneven scenes processed together, forward and backward
        _case("batch12_step_bf16", "batch", "bf16", 64, 512, 896, 1800, scenes=12),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["forward", "forward", "train", "train", "train", "frame_fp8", "fused",
                       "batch"])
    dtype = "f32" if kind == "frame_fp8" else rng.choice(["f32", "bf16", "bf16", "f16"])
    channels, groups = rng.choice([(64, 4), (128, 4), (256, 8), (256, 8)])
    img_h, img_w = rng.choice([(128, 224), (256, 448), (256, 704), (270, 492), (384, 640)])
    cams = _log_int(rng, 2, 64)
    anchors = _log_int(rng, 100, 1800)
    points = rng.choice([7, 11, 13])
    levels = rng.choice([3, 4, 4])
    batch = rng.choice([1, 1, 2]) if kind in ("forward", "train") else 1
    scenes = rng.randint(2, 5) if kind == "batch" else 1
    # no more samples in all than twice the 64-camera scene's
    anchors = max(50, min(anchors, 6_000_000 // (batch * scenes * cams * points * levels)))
    out_of_view = 0.0 if kind in ("fused", "batch") else rng.choice([0.0, 0.25])
    return _case(None, kind, dtype, cams, img_h, img_w, anchors, batch=batch, levels=levels,
                 channels=channels, groups=groups, points=points, out_of_view=out_of_view,
                 logits=kind != "frame_fp8" and rng.random() < 0.3, scenes=scenes,
                 mixed=kind != "fused" and rng.random() < 0.3)


# ------------------------------------------------------------------ inputs

def _scenes(c):
    """(cams, (img_h, img_w), anchors) of each scene."""
    if c["kind"] != "batch":
        return [(c["cams"], (c["img_h"], c["img_w"]), c["anchors"])]
    # the uneven batch: camera counts, image sizes and anchors as synth draws them,
    # within the case's largest
    return [(min(n, c["cams"]), (min(h, c["img_h"]), min(w, c["img_w"])), min(a, c["anchors"]))
            for n, (h, w), a in synth.batched_scene_shapes(0, c["scenes"])]


def _geometry(c, cams, img):
    """(spatial_shapes, level_start_index, rows); with `mixed`, the cameras'
    images differ in size."""
    levels = []
    for n in range(cams):
        h, w = img if not c["mixed"] else (img[0] - 13 * (n % 3), img[1] - 21 * (n % 4))
        levels.append([(max(1, h // s), max(1, w // s)) for s in STRIDES[:c["levels"]]])
    return synth.layout(levels)


def _randn(gen, *shape):
    return torch.randn(*shape, generator=gen, device="cuda")


def _rand(gen, *shape):
    return torch.rand(*shape, generator=gen, device="cuda")


def _locations(c, gen, B, A, N):
    P = c["points"]
    loc = _rand(gen, B, A, P, N, 2) * 1.1 - 0.05
    if c["out_of_view"]:
        # out of view: a band beyond every level along one axis
        out = _rand(gen, B, A, P, N) < c["out_of_view"]
        band = 0.5 * _rand(gen, B, A, P, N)
        side = torch.where(_rand(gen, B, A, P, N) < 0.5, -1.0 + band, 1.5 + band)
        axis = _rand(gen, B, A, P, N) < 0.5
        loc[..., 0] = torch.where(out & axis, side, loc[..., 0])
        loc[..., 1] = torch.where(out & ~axis, side, loc[..., 1])
    return loc.contiguous()


def _weights(c, gen, B, A, N):
    P, L, G = c["points"], c["levels"], c["groups"]
    x = _randn(gen, B, A, P * N * L, G)
    x = 2.0 * x if c["logits"] else torch.softmax(x, dim=2)
    return x.reshape(B, A, P, N, L, G).contiguous()


def _project64(anchors, keypoints, projection, image_hw, dt):
    """float64 (locations [B, A, P, N, 2], visible [B, A, N], distance in
    pixels of each anchor's nearest keypoint to an image border or the focal
    plane [B, A])."""
    a, k, m = anchors.double(), keypoints.double(), projection.double()
    c, s = torch.cos(a[..., 6:7]), torch.sin(a[..., 6:7])
    o = k * a[:, :, None, 3:6]
    world = torch.stack([c * o[..., 0] - s * o[..., 1], s * o[..., 0] + c * o[..., 1], o[..., 2]],
                        dim=-1)
    world = world + (a[..., 0:3] + dt * a[..., 7:10])[:, :, None]
    ones = torch.ones_like(world[..., :1])
    p = (torch.cat([world, ones], -1)[:, :, :, None, None, :] * m[:, None, None]).sum(-1)
    depth = p[..., 2]
    front = depth > 1e-5
    pix = p[..., :2] / torch.where(front, depth, torch.ones_like(depth))[..., None]
    size = image_hw.double().flip(-1)                      # (W, H)
    inside = front[..., None] & (pix >= 0) & (pix < size)
    border = torch.minimum(pix.abs(), (pix - size).abs()).amin(-1)
    near = torch.where(front, border, (depth - 1e-5).abs() * 1e3)
    loc = torch.where(front[..., None], pix / size, torch.full_like(pix, -2.0))
    return loc, inside.all(-1).any(2), near.amin(3).amin(2)


def _outside_in(c, gen, seed):
    """The outside-in network's geometry, anchors whose keypoints fall within
    0.02 px of an image border moved (their visibility would be a matter of
    rounding)."""
    g = synth.outside_in(seed, 1, c["cams"], c["anchors"], c["points"], (c["img_h"], c["img_w"]))
    a, k, m, hw = (t.cuda() for t in (g.anchors, g.keypoints, g.projection, g.image_hw))
    for _ in range(50):
        near = _project64(a, k, m, hw, g.dt)[2] < 0.02
        if not bool(near.any()):
            break
        a[..., :2] = torch.where(near[..., None], (2 * _rand(gen, 1, c["anchors"], 2) - 1) * 30,
                                 a[..., :2])
    return a.contiguous(), k, m, hw, g.dt


def _inputs(c, seed):
    """One dict of device tensors per scene, from the seed alone."""
    gen = torch.Generator("cuda").manual_seed(seed)
    found = []
    for cams, img, A in _scenes(c):
        shapes, starts, rows = _geometry(c, cams, img)
        B, C = c["batch"], c["channels"]
        x = dict(shapes=shapes, starts=starts,
                 feat=_randn(gen, B, rows, C).to(DTYPES[c["dtype"]]),
                 w=_weights(c, gen, B, A, cams))
        if c["kind"] == "fused":
            x["geometry"] = _outside_in(c, gen, seed)
            x["score"] = _rand(gen, B, A, cams) + 0.05
        else:
            x["loc"] = _locations(c, gen, B, A, cams)
        if c["kind"] in ("train", "fused", "batch"):
            x["go"] = _randn(gen, B, A, C)
        found.append(x)
    return found


def prepare(case, seed):
    c, xs = case, _inputs(case, seed)
    s = {"case": c}
    if c["kind"] == "batch":
        s["go"] = [x["go"][0] for x in xs]
        s["batch"] = ops.SceneBatch(
            [(x["feat"][0], ops.Layout(x["shapes"], x["starts"]), x["loc"][0], x["w"][0])
             for x in xs], logits=c["logits"])
        return s
    s.update(xs[0], layout=ops.Layout(xs[0]["shapes"], xs[0]["starts"]))
    if c["kind"] == "train":
        for k in ("feat", "loc", "w"):
            s[k].requires_grad_(True)
    return s


# ------------------------------------------------------------------ one pass

def run(state):
    s = state
    c = s["case"]
    kind, logits = c["kind"], c["logits"]
    if kind == "forward":
        return {"out": ops.forward(s["feat"], s["layout"], s["loc"], s["w"], logits=logits)}
    if kind == "frame_fp8":
        codes, scale = ops.quantize_fp8(s["feat"], s["layout"])
        out = ops.forward(codes, s["layout"], s["loc"], s["w"], level_scale=scale, logits=logits)
        return {"codes": codes, "scale": scale, "out": out}
    if kind == "train":
        leaves = (s["feat"], s["loc"], s["w"])
        out = ops.msda(s["feat"], s["layout"], s["loc"], s["w"], logits=logits)
        gf, gl, gw = torch.autograd.grad(out, leaves, s["go"])
        return {"out": out, "grad_feat": gf, "grad_loc": gl, "grad_w": gw}
    if kind == "fused":
        loc, visible = ops.project_keypoints(*s["geometry"])
        out = ops.forward_fused(s["feat"], s["layout"], loc, s["w"], visible, s["score"],
                                logits=logits)
        gf, gl, gw, gs = ops.backward_fused(s["feat"], s["layout"], loc, s["w"], visible,
                                            s["score"], out, s["go"], logits=logits)
        return {"loc": loc, "visible": visible, "out": out, "grad_feat": gf, "grad_loc": gl,
                "grad_w": gw, "grad_score": gs}
    b = s["batch"]
    out = b.forward()
    torch._foreach_copy_(b.grad_out, s["go"])
    gf, gl, gw = b.backward()
    return {"out": out, "grad_feat": gf, "grad_loc": gl, "grad_w": gw}


def work(case):
    """Bytes: every input read once, every output written once. Operations: 8
    per (sample, channel) for the forward's interpolation, 8 each for the
    backward's corner products and grad_feat contributions."""
    c = case
    L, C, G, P, B = c["levels"], c["channels"], c["groups"], c["points"], c["batch"]
    step = c["kind"] in ("train", "fused", "batch")
    eb = 4 if c["dtype"] == "f32" else 2
    nbytes = flops = 0
    for cams, img, A in _scenes(c):
        rows = _geometry(c, cams, img)[2]
        pairs = B * A * P * cams
        samples = pairs * L
        feat = B * rows * C
        nbytes += feat * eb + samples * G * 4 + pairs * 8 + B * A * C * 4
        flops += 8 * samples * C
        if c["kind"] == "frame_fp8":
            nbytes += feat
        if step:
            nbytes += feat * eb + samples * G * 4 + pairs * 8 + B * A * C * 4
            flops += 16 * samples * C
        if c["kind"] == "fused":
            nbytes += B * A * cams * 9 + B * A * (10 + 3 * P) * 4
    return {"bytes": nbytes, "flops": flops}


# ------------------------------------------------------------------ float64

def _quantised(x, shapes, starts):
    """(scale [L], dequantised float64 features) of the per-level e4m3 form."""
    L = shapes.shape[1]
    spans = [[(int(starts[n, l]), int(starts[n, l] + shapes[n, l, 0] * shapes[n, l, 1]))
              for n in range(shapes.shape[0])] for l in range(L)]
    scale, deq = [], torch.zeros(x.shape, dtype=torch.float64, device=x.device)
    for per_cam in spans:
        amax = max(float(x[:, i:j].abs().max()) for i, j in per_cam)
        s = torch.tensor(amax, dtype=torch.float32, device=x.device) / 448.0
        s = torch.where(s == 0, torch.ones_like(s), s)
        for i, j in per_cam:
            q = (x[:, i:j] / s).clamp(-448, 448).to(torch.float8_e4m3fn)
            deq[:, i:j] = q.to(torch.float32).double() * s.double()
        scale.append(s.double())
    return torch.stack(scale), deq


def _msda64(feat, shapes, starts, loc, w, go=None, view=None):
    """(out, grad_feat, grad_loc, grad_w, grad_view) in float64 over one
    batch item: feat [R, C], loc [A, P, N, 2], w [A, P, N, L, G], go [A, C] or
    None, view [A, N] factors of the cameras (None: 1). Anchors in chunks."""
    A, P, N, L, G = w.shape
    R, C = feat.shape
    H = shapes[..., 0].to(feat.device).double()
    W = shapes[..., 1].to(feat.device).double()
    first = starts.to(feat.device).long()
    view = torch.ones(A, N, dtype=torch.float64, device=feat.device) if view is None else view
    out = torch.zeros(A, C, dtype=torch.float64, device=feat.device)
    gf = torch.zeros_like(feat) if go is not None else None
    gl, gw, gv = torch.zeros_like(loc), torch.zeros_like(w), torch.zeros_like(view)
    chunk = max(1, int(4e8 // (P * N * L * 4 * C)))
    for a0 in range(0, A, chunk):
        a1 = min(A, a0 + chunk)
        n = a1 - a0
        x = loc[a0:a1, ..., 0:1] * W - 0.5                   # [n, P, N, L]
        y = loc[a0:a1, ..., 1:2] * H - 0.5
        live = (x > -1) & (x < W) & (y > -1) & (y < H)
        x0, y0 = torch.floor(x), torch.floor(y)
        lx, ly = x - x0, y - y0
        rows, cw, dx, dy = [], [], [], []
        for j in (0, 1):
            for i in (0, 1):
                xi, yj = x0 + i, y0 + j
                ok = live & (xi >= 0) & (xi < W) & (yj >= 0) & (yj < H)
                rows.append(torch.where(ok, first + (yj * W + xi).long(), -1))
                fx, fy = (lx if i else 1 - lx), (ly if j else 1 - ly)
                cw.append(fx * fy)
                dx.append((1 if i else -1) * fy * W)
                dy.append((1 if j else -1) * fx * H)
        rows = torch.stack(rows, -1)                         # [n, P, N, L, 4]
        inside = (rows >= 0).double()
        cw, dx, dy = (torch.stack(t, -1) * inside for t in (cw, dx, dy))
        rows = rows.clamp(min=0).reshape(-1)
        F = feat[rows].reshape(n, -1, 4, G, C // G)
        wc = w[a0:a1] * view[a0:a1, None, :, None, None]
        wf = wc.reshape(n, -1, G)
        cwf = cw.reshape(n, -1, 4)
        out[a0:a1] = ((F * cwf[..., None, None]).sum(2) * wf[..., None]).sum(1).reshape(n, C)
        if go is None:
            continue
        g = go[a0:a1].reshape(n, 1, 1, G, C // G)
        d = (F * g).sum(-1)                                  # [n, S, 4, G]
        del F
        dw = (d * cwf[..., None]).sum(2).reshape(n, P, N, L, G)
        gw[a0:a1] = dw * view[a0:a1, None, :, None, None]
        gv[a0:a1] = (dw * w[a0:a1]).sum((1, 3, 4))
        dc = (d * wf[:, :, None, :]).sum(-1).reshape(n, P, N, L, 4)
        gl[a0:a1, ..., 0] = (dc * dx).sum((-1, -2))
        gl[a0:a1, ..., 1] = (dc * dy).sum((-1, -2))
        k = cwf[..., None, None] * wf[:, :, None, :, None] * g
        gf.index_add_(0, rows, k.reshape(-1, C))
    return out, gf, gl, gw, gv


def exact(case, seed):
    c = case
    outs = []
    for x in _inputs(c, seed):
        B, A, G = c["batch"], x["w"].shape[1], c["groups"]
        scale = vis = loc64 = None
        feat = x["feat"]
        if c["kind"] == "frame_fp8":
            scale, feat = _quantised(feat, x["shapes"], x["starts"])
        if c["kind"] == "fused":
            loc64, vis, _ = _project64(*x["geometry"])
        r = {k: [] for k in ("out", "grad_feat", "grad_loc", "grad_w", "grad_score")}
        for b in range(B):
            raw = x["w"][b].double()
            w = torch.softmax(raw.reshape(A, -1, G), 1).reshape(raw.shape) if c["logits"] else raw
            loc = (x["loc"] if loc64 is None else loc64)[b].double()
            go = x["go"][b].double() if "go" in x else None
            view = None
            if vis is not None:
                score = x["score"][b].double() * vis[b]
                V = score.sum(-1, keepdim=True)
                view = torch.where(V > 0, score / torch.where(V > 0, V, torch.ones_like(V)),
                                   torch.zeros_like(score))
            o, gf, gl, gw, gv = _msda64(feat[b].double(), x["shapes"], x["starts"], loc, w, go, view)
            r["out"].append(o)
            if go is None:
                continue
            if c["logits"]:
                gw = w * (gw - (w * gw).reshape(A, -1, G).sum(1)[:, None, None, None, :])
            if vis is not None:
                dot = (go * o).sum(-1, keepdim=True)
                r["grad_score"].append(torch.where(vis[b] & (V > 0), (gv - dot) / V.clamp(min=1e-30),
                                                   torch.zeros_like(gv)))
            for k, t in (("grad_feat", gf), ("grad_loc", gl), ("grad_w", gw)):
                r[k].append(t)
        outs.append(({k: torch.stack(v) for k, v in r.items() if v}, scale, loc64))
    if c["kind"] == "batch":
        return {k: [o[k][0] for o, _, _ in outs] for k in ("out", "grad_feat", "grad_loc", "grad_w")}
    found, scale, loc64 = outs[0]
    if c["kind"] == "frame_fp8":
        return {"codes": None, "scale": scale, "out": found["out"]}
    if c["kind"] == "fused":
        return dict(found, loc=loc64, visible=None)
    return found
