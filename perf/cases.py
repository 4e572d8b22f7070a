"""What a user of the engine has it do, as timed cases: detection at one exit, every exit in one pass, mixed plans, and the
image classifier, from one small frame to a 256-frame video.

The detectors and the classifier are those of thia_synth.CONFIGS and thia_synth.VGG16_EXITS (random weights with the gains
of thia_synth.recipe_for); frames are synthetic traffic-camera scenes (shaded road, moving solid rectangles, sensor noise)
drawn on the GPU from the seed.  One model of each kind is resident per process, as in the engine's own use: many videos,
one model.
"""
import math
import random
from dataclasses import replace

import numpy as np
import torch

import paper_2102_08481_amd as thia
from thia_synth import CONFIGS, VGG16_EXITS, recipe_for
from thia_synth.classifier import classifier_tensor_list
from thia_synth.weights import tensor_list

# model name -> (specification, rectangles per scene (least, most), their longer side in pixels (least, most))
DETECTORS = {
    "tiny-fp32": (CONFIGS[1].model, (3, 6), (12, 64)),
    "r50": (CONFIGS[3].model, (5, 40), (16, 300)),
    "r50-fp32": (replace(CONFIGS[3].model, precision=0), (5, 40), (16, 300)),
    "r101": (CONFIGS[5].model, (20, 150), (8, 400)),
}
CLASSIFIERS = {"vgg16": VGG16_EXITS, "vgg16-fp32": replace(VGG16_EXITS, precision=0)}


def listed():
    return [
        # the smallest call: four thumbnails through the one-exit fp32 detector; launches and latency are all there is
        {"name": "tiny-fp32", "kind": "detect", "model": "tiny-fp32", "n": 4, "H": 128, "W": 128, "ep": 1},
        # a live camera, frame by frame: the first exit for an easy scene, the last for a hard one
        {"name": "live-ep1", "kind": "detect", "model": "r50", "n": 1, "H": 540, "W": 960, "ep": 1},
        {"name": "live-ep4", "kind": "detect", "model": "r50", "n": 1, "H": 540, "W": 960, "ep": 4},
        # a short chunk of an odd-sized stream: ragged tiles everywhere, rows that start on odd addresses
        {"name": "odd-ep3", "kind": "detect", "model": "r50", "n": 5, "H": 361, "W": 643, "ep": 3},
        # ordinary chunks of stored video at the exits a planner picks
        {"name": "chunk16-ep2", "kind": "detect", "model": "r50", "n": 16, "H": 540, "W": 960, "ep": 2},
        {"name": "chunk32-ep1", "kind": "detect", "model": "r50", "n": 32, "H": 540, "W": 960, "ep": 1},
        {"name": "chunk32-ep4", "kind": "detect", "model": "r50", "n": 32, "H": 540, "W": 960, "ep": 4},
        # the planner scores every exit on a batch of sampled frames
        {"name": "all-exits16", "kind": "all_exits", "model": "r50", "n": 16, "H": 540, "W": 960},
        # a planned query's execution: 256 frames, eight chunks at mixed exits
        {"name": "plan-8x32", "kind": "plan", "model": "r50", "chunk": 32, "plan": "1,4,2,2,3,1,4,3", "H": 540, "W": 960},
        # full-HD chunk through the deep backbone, 2000 proposals in front of the suppression and 20 classes
        {"name": "hd-r101-ep4", "kind": "detect", "model": "r101", "n": 8, "H": 1080, "W": 1920, "ep": 4},
        # single-precision detection, for users who compare against a single-precision reference
        {"name": "fp32-ep2", "kind": "detect", "model": "r50-fp32", "n": 2, "H": 540, "W": 960, "ep": 2},
        # a batch of pictures through the classifier's last exit
        {"name": "classify64", "kind": "classify", "model": "vgg16", "n": 64, "H": 224, "W": 224, "ep": 8},
    ]


def _between(rng, low, high):
    """A whole number from low to high, spread over its logarithm."""
    return min(high, max(low, int(math.exp(rng.uniform(math.log(low), math.log(high + 1))))))


def draw(rng):
    kind = rng.choices(["detect", "all_exits", "plan", "classify"], [6, 1, 2, 1])[0]
    if kind == "classify":
        model = rng.choice(["vgg16", "vgg16", "vgg16-fp32"])
        n = _between(rng, 1, 64 if model == "vgg16" else 8)
        return {"kind": kind, "model": model, "n": n, "H": _between(rng, 96, 300), "W": _between(rng, 96, 300), "ep": rng.randint(1, 8)}
    model = "r50" if kind != "detect" else rng.choices(["r50", "r101", "r50-fp32", "tiny-fp32"], [6, 2, 1, 1])[0]
    if model == "tiny-fp32":
        return {"kind": kind, "model": model, "n": _between(rng, 1, 16), "H": _between(rng, 64, 256), "W": _between(rng, 64, 256), "ep": 1}
    H = _between(rng, 128, 1080)
    W = int(H * rng.uniform(1.2, 1.9))
    # frames that fit the case's share of pixels: the 32-frame chunk's, for single precision two frames'
    most = {"r50-fp32": 2, "r101": 24}.get(model, 32) * 540 * 960 // (H * W)
    n = _between(rng, 1, max(1, min(32, most)))
    if kind == "plan":
        chunks = rng.randint(2, 8)
        return {"kind": kind, "model": model, "chunk": n, "plan": ",".join(str(rng.randint(0, 4)) for _ in range(chunks - 1)) + ",%d" % rng.randint(1, 4),
                "H": H, "W": W}
    case = {"kind": kind, "model": model, "n": n, "H": H, "W": W}
    if kind == "detect":
        case["ep"] = rng.randint(1, 4)
    return case


# ---------------------------------------------------------------------------------------------------- resident models
_resident = {}


def _blob(spec, tensors, gains):
    """The weights blob of `spec`, its normal values drawn on the GPU: std sqrt(2 / fan_in) and the recipe's gains."""
    gen = torch.Generator(device="cuda").manual_seed(20481)
    parts = [np.frombuffer(spec.header(), dtype=np.uint8)]
    for _, shape, role in tensors:
        size = math.prod(shape)
        if role == "bias":
            parts.append(np.zeros(4 * size, np.uint8))
            continue
        std = {"pred": gains["pred_std"], "pred_delta": gains.get("delta_std")}.get(role) or math.sqrt(2.0 / math.prod(shape[1:]))
        if role == "res_last":
            std *= gains["res_gain"]
        parts.append((torch.randn(size, generator=gen, device="cuda") * std).cpu().numpy().view(np.uint8))
    return np.concatenate(parts)


def _model(name):
    if name not in _resident:
        if name in CLASSIFIERS:
            spec = CLASSIFIERS[name]
            _resident[name] = thia.thia_classifier_load(_blob(spec, classifier_tensor_list(spec), {"pred_std": 0.05}), spec.n_exits)
        else:
            spec = DETECTORS[name][0]
            _resident[name] = thia.thia_load_model(_blob(spec, tensor_list(spec), recipe_for(spec)), spec.n_exits)
    return _resident[name]


# ------------------------------------------------------------------------------------------------------------- inputs
def _scene(n, H, W, seed, rects, sides, pictures):
    """uint8 [n,3,H,W]: a shaded background with rectangles that move from frame to frame (`pictures`: every frame a scene of
    its own), and sensor noise of up to 16 grey levels."""
    r = random.Random(seed)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    y = torch.arange(H, device="cuda", dtype=torch.float32)[:, None] / H
    x = torch.arange(W, device="cuda", dtype=torch.float32)[None, :] / W

    def background():
        shade = 8 * torch.cos(6.2832 * (r.random() * x + r.random() * y + r.random())) + 5 * torch.cos(6.2832 * (1.7 * r.random() * x - 1.3 * r.random() * y))
        base = 100 + 30 * r.random()
        level = [r.uniform(20, 230) if pictures else base + 3 * (r.random() - 0.5) for _ in range(3)]
        return torch.stack([c + shade for c in level]).round().clamp(0, 255).to(torch.uint8)

    def rectangles():
        got = []
        for _ in range(r.randint(*rects)):
            side, aspect, angle, speed = r.uniform(*sides), r.uniform(0.5, 2.5), r.uniform(0, 6.2832), r.uniform(1, 4)
            w, h = (side, side / aspect) if aspect >= 1 else (side * aspect, side)
            colour = torch.tensor([r.randrange(256) for _ in range(3)], dtype=torch.uint8, device="cuda")[:, None, None]
            got.append((r.random() * W, r.random() * H, speed * math.cos(angle), speed * math.sin(angle), max(2, int(w)), max(2, int(h)), colour))
        return got

    frames = torch.empty((n, 3, H, W), dtype=torch.uint8, device="cuda")
    scene = None
    for t in range(n):
        if scene is None or pictures:
            scene = background(), rectangles()
        frames[t] = scene[0]
        for cx, cy, vx, vy, w, h, colour in scene[1]:
            x0, y0 = int((cx + vx * t) % W - w / 2), int((cy + vy * t) % H - h / 2)
            frames[t, :, max(y0, 0):max(y0 + h, 0), max(x0, 0):max(x0 + w, 0)] = colour
    for t in range(0, n, 32):
        part = frames[t:t + 32]
        noise = torch.randint(-16, 17, part.shape, generator=gen, device="cuda", dtype=torch.int16)
        part.copy_((part.to(torch.int16) + noise).clamp_(0, 255))
    return frames


def _frames_of(case):
    return case["chunk"] * len(case["plan"].split(",")) if case["kind"] == "plan" else case["n"]


def prepare(case, seed):
    rects, sides = DETECTORS[case["model"]][1:] if case["model"] in DETECTORS else ((3, 12), (12, 120))
    frames = _scene(_frames_of(case), case["H"], case["W"], seed, rects, sides, case["kind"] == "classify")
    state = dict(case, loaded=_model(case["model"]), frames=frames)
    if case["kind"] == "plan":
        state["plan"] = [int(e) for e in case["plan"].split(",")]
    return state


def run(state):
    m, frames = state["loaded"], state["frames"]
    if state["kind"] == "classify":
        labels, conf, logits = thia.thia_classify_chunk(m, frames, state["ep"], want_logits=True)
        return {"labels": labels, "conf": conf, "logits": logits}
    if state["kind"] == "all_exits":
        boxes, scores, labels = thia.thia_detect_all_exits(m, frames)
    elif state["kind"] == "plan":
        boxes, scores, labels = thia.thia_run_plan(m, frames, state["chunk"], state["plan"])
    else:
        boxes, scores, labels = thia.thia_detect_chunk(m, frames, state["ep"])
    return {"boxes": boxes, "scores": scores, "labels": labels}


# --------------------------------------------------------------------------------------------------------------- work
def _half(v):
    return (v - 1) // 2 + 1   # output size of the stride-2 layers: 7x7 pad 3, 3x3 pad 1


def _detector_macs(spec, H, W, exits):
    """(multiply-adds per frame, weight elements) of one backbone pass to the deepest of `exits` with the units of each."""
    h, w = _half(H), _half(W)
    macs = h * w * spec.stem_ch * 147
    params = spec.stem_ch * 147
    h, w = _half(h), _half(w)
    cin = spec.stem_ch
    for s in range(max(exits)):
        wd = spec.base_width << s
        for b in range(spec.blocks[s]):
            ho, wo = (_half(h), _half(w)) if b == 0 and s > 0 else (h, w)
            short = cin * 4 * wd if b == 0 else 0
            macs += h * w * cin * wd + ho * wo * (9 * wd * wd + 4 * wd * wd + short)
            params += cin * wd + 9 * wd * wd + 4 * wd * wd + short
            cin, h, w = 4 * wd, ho, wo
        if s + 1 in exits:
            hc = spec.head_ch if spec.has_lateral else cin
            rpn = (cin * hc if spec.has_lateral else 0) + 9 * hc * hc + 5 * spec.n_anchors * hc
            box = hc * spec.pool ** 2 * spec.fc_dim + spec.fc_dim ** 2 + 5 * spec.n_classes * spec.fc_dim
            macs += h * w * rpn + spec.post_nms * box
            params += rpn + box
    return macs, params


def work(case):
    n, pixels = _frames_of(case), case["H"] * case["W"]
    if case["kind"] == "classify":
        spec = CLASSIFIERS[case["model"]]
        h, w, cin, macs, params = case["H"], case["W"], spec.in_ch, 0, 0
        tap = spec.taps[case["ep"] - 1]
        for i in range(tap):
            macs += h * w * 9 * cin * spec.channels[i]
            params += 9 * cin * spec.channels[i]
            cin = spec.channels[i]
            if i + 1 in spec.pool_after:
                h, w = h // 2, w // 2
        macs, params = macs + cin * spec.n_classes, params + cin * spec.n_classes
        return {"bytes": 3 * pixels * n + params * (2 if spec.precision else 4) + n * 4 * (2 + spec.n_classes), "flops": 2 * macs * n}
    spec = DETECTORS[case["model"]][0]
    out = n * spec.max_det * 24
    if case["kind"] == "plan":
        plan = [int(e) for e in case["plan"].split(",")]
        macs = sum(case["chunk"] * _detector_macs(spec, case["H"], case["W"], [e])[0] for e in plan if e)
        params = _detector_macs(spec, case["H"], case["W"], sorted(set(plan) - {0}))[1]
        n = case["chunk"] * sum(e > 0 for e in plan)
    else:
        exits = range(1, spec.n_exits + 1) if case["kind"] == "all_exits" else [case["ep"]]
        macs, params = _detector_macs(spec, case["H"], case["W"], exits)
        macs, out = macs * n, out * len(exits)
    return {"bytes": 3 * pixels * n + params * (2 if spec.precision else 4) + out, "flops": 2 * macs}


def tolerance(case):
    """Largest error of the values, and the share of labels that a tie may turn.  Measured: the detectors' kernels, fused or
    layer by layer, give the same lists bit for bit at every batch size; the classifier's logits and confidences in bf16 are
    2.4e-3 and 5.4e-3 from those of the fp32 model; fp32 sums taken in another order move logits by 2e-6."""
    if case["model"] in CLASSIFIERS:
        return {"rel": 2e-2 if CLASSIFIERS[case["model"]].precision else 1e-5, "differ": 0.01}
    return {"rel": 1e-2 if DETECTORS[case["model"]][0].precision else 1e-5, "differ": 0.01}
