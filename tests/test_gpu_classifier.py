"""The image classifier with exits (the paper's generalisation of early inference, Sec. 4.2) on the GPU against its CPU
oracle, through the C ABI: single steps on identical inputs, every exit of a reduced network element by element, and the
full VGG-16-style network (thirteen 3x3 layers, eight exits, 102 classes) at 224 x 224."""
import numpy as np
import pytest
import torch

from gpu_common import MINI_BF16, gpu_model, nchw_to_nhwc, relerr, to_dev
from oracle import classifier as oc
from thia_synth import ClassifierSpec, VGG16_EXITS, SceneSpec, make_classifier_blob, make_frames, split_classifier_blob

pytestmark = pytest.mark.gpu

TOL = {0: 1e-4, 1: 2e-2}      # logits, per tensor max |gpu - ref| / max |ref|: fp32 path; bf16 path vs the fp32 oracle
SMALL = {p: ClassifierSpec(precision=p, channels=(64, 64, 128, 128, 192), pool_after=(2, 4), taps=(1, 2, 4, 5), n_classes=11) for p in (0, 1)}
_cache = {}


def _clf(spec, seed):
    from paper_2102_08481_amd import thia_classifier_load
    key = (spec.header(), seed)
    if key not in _cache:
        blob = make_classifier_blob(spec, seed)
        _cache[key] = (thia_classifier_load(blob, spec.n_exits), blob)
    return _cache[key]


def _check_answers(labels, conf, logits, ref, tol):
    """Logits within tol; where the reference's best class leads the runner-up by more than the error bound both sides must
    name it (the decision is then not a matter of rounding); elsewhere the GPU's label must be one of the near-tied classes."""
    g_lab, g_conf, g_log = labels.cpu().numpy(), conf.cpu().numpy(), logits.cpu().numpy()
    err = relerr(g_log, ref["logits"])
    assert err <= tol, err
    bound = 2 * tol * np.max(np.abs(ref["logits"]))
    srt = np.sort(ref["logits"], axis=1)
    clear = srt[:, -1] - srt[:, -2] > bound
    assert np.array_equal(g_lab[clear], ref["labels"][clear])
    for f in np.flatnonzero(~clear):
        assert ref["logits"][f, g_lab[f]] >= srt[f, -1] - bound
    assert np.array_equal(g_lab, np.argmax(g_log, axis=1))            # the GPU's own decision: first maximum of its own logits
    assert np.max(np.abs(g_conf[clear] - ref["conf"][clear])) <= 4 * bound + 1e-5
    return err, int(clear.sum())


@pytest.mark.parametrize("precision", [0, 1])
def test_pool_step_matches_oracle(precision):
    c, _ = _clf(SMALL[precision], 70)
    rs = np.random.RandomState(1)
    for (n, H, W, C) in [(2, 8, 8, 64), (3, 9, 11, 64), (1, 33, 20, 192)]:
        x = rs.randn(n, C, H, W).astype(np.float32)
        if precision:
            x = torch.from_numpy(x).to(torch.bfloat16).float().numpy()
        y = c.op_pool(to_dev(nchw_to_nhwc(x), c.elem))
        torch.cuda.synchronize()
        assert np.array_equal(y.float().cpu().numpy(), nchw_to_nhwc(oc.maxpool2x2(x)))       # a maximum is exact


@pytest.mark.parametrize("precision", [0, 1])
def test_unit_step_matches_oracle(precision):
    """Global average pooling + FC + soft-max + arg-max on the oracle's tapped tensor (teacher forcing)."""
    spec = SMALL[precision]
    c, blob = _clf(spec, 70)
    fr = make_frames(SceneSpec(45, 61, 3, 2, 4, 8, 30, "gradient"), 5)
    for ep in (1, 4):
        ref = oc.classify(blob, fr, ep)
        n, C, h, w = ref["feat"].shape
        feat = to_dev(nchw_to_nhwc(ref["feat"]).reshape(n, h * w, C), c.elem)
        lab, conf, log = c.op_unit(feat, ep)
        torch.cuda.synchronize()
        _check_answers(lab, conf, log, ref, 1e-5)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("ep", [0, 1, 2, 3, 4])
def test_small_classifier_every_exit(precision, ep):
    spec = SMALL[precision]
    c, blob = _clf(spec, 70)
    fr = make_frames(SceneSpec(45, 61, 5, 2, 4, 8, 30, "gradient"), 6)       # odd sizes: ragged tiles, dropped pool rows
    lab, conf, log = c.classify_chunk(to_dev(fr), ep, want_logits=True)
    torch.cuda.synchronize()
    if ep == 0:
        assert (lab == -1).all() and (conf == 0).all()
        return
    ref = oc.classify(blob, fr, ep, precision=0)
    err, n_clear = _check_answers(lab, conf, log, ref, TOL[precision])
    print(f"small classifier precision {precision} exit {ep}: logits max rel err {err:.2e}, {n_clear}/5 decisions beyond rounding")
    # the same call again is bit-identical, and a frame's answer does not depend on its chunk
    lab2, conf2, log2 = c.classify_chunk(to_dev(fr[1:3]), ep, want_logits=True)
    torch.cuda.synchronize()
    assert torch.equal(log2, log[1:3]) and torch.equal(lab2, lab[1:3]) and torch.equal(conf2, conf[1:3])


def test_exits_stop_early_and_share_the_prefix():
    """Layers behind the tapped one are not run (changed weights there change nothing), which is early inference."""
    spec = SMALL[1]
    blob = make_classifier_blob(spec, 70)
    poisoned = blob.copy()
    t = split_classifier_blob(spec, poisoned)
    for i in range(spec.taps[1] + 1, spec.n_layers + 1):
        t[f"conv{i}.w"][...] = 0.5
    from paper_2102_08481_amd import thia_classifier_load
    c, _ = _clf(spec, 70)
    cp = thia_classifier_load(poisoned, spec.n_exits)
    fr = to_dev(make_frames(SceneSpec(45, 61, 2, 2, 4, 8, 30, "gradient"), 8))
    a = c.classify_chunk(fr, 2, want_logits=True)
    b = cp.classify_chunk(fr, 2, want_logits=True)
    torch.cuda.synchronize()
    assert torch.equal(a[2], b[2]) and torch.equal(a[0], b[0])
    a3 = c.classify_chunk(fr, 3, want_logits=True)[2]
    b3 = cp.classify_chunk(fr, 3, want_logits=True)[2]
    torch.cuda.synchronize()
    assert not torch.equal(a3, b3)                     # (the changed layers do matter one exit further on)
    cp.close()


@pytest.mark.parametrize("ep", [1, 4, 8])
def test_vgg16_eight_exits_at_224(ep):
    """The paper's generalisation case at its real shape: VGG-16's thirteen layers, eight exits, 102 classes, 224 x 224 frames,
    bf16; the oracle is run on the first two frames of an 8-frame chunk."""
    spec = VGG16_EXITS
    c, blob = _clf(spec, 71)
    fr = make_frames(SceneSpec(224, 224, 8, 3, 8, 16, 120, "gradient"), 9)
    lab, conf, log = c.classify_chunk(to_dev(fr), ep, want_logits=True)
    torch.cuda.synchronize()
    assert ((lab >= 0) & (lab < 102)).all() and ((conf > 0) & (conf <= 1)).all()
    ref = oc.classify(blob, fr[:2], ep, precision=0)
    err, n_clear = _check_answers(lab[:2], conf[:2], log[:2], ref, TOL[1])
    print(f"VGG-16-style exit {ep}: logits max rel err vs fp32 oracle {err:.2e}, {n_clear}/2 decisions beyond rounding")


def test_classifier_argument_errors():
    from paper_2102_08481_amd import ThiaError, thia_classifier_load
    spec = SMALL[1]
    c, blob = _clf(spec, 70)
    fr = to_dev(make_frames(SceneSpec(45, 61, 1, 2, 4, 8, 30, "gradient"), 8))
    with pytest.raises(ThiaError) as e:
        c.classify_chunk(fr, 5)
    assert e.value.code == -2
    with pytest.raises(ThiaError) as e:
        thia_classifier_load(blob[:-4], spec.n_exits)
    assert e.value.code == -4
    with pytest.raises(ThiaError) as e:
        thia_classifier_load(blob, spec.n_exits + 1)
    assert e.value.code == -4
    tiny = to_dev(np.zeros((1, 3, 1, 1), np.uint8))
    with pytest.raises(ThiaError) as e:
        c.classify_chunk(tiny, 4)                      # two pools in front of exit 4 leave no position
    assert e.value.code == -3
    lab, conf = c.classify_chunk(tiny, 1)              # exit 1 has no pool in front of it
    torch.cuda.synchronize()
    assert 0 <= int(lab[0]) < spec.n_classes


@pytest.mark.parametrize("channels,pools", [((64, 64, 64), (2,)), ((64, 64, 64), (1, 2)), ((128, 64, 64), (1,)), ((64, 128, 64), ())])
@pytest.mark.parametrize("n,H,W", [(3, 4, 5), (2, 16, 32), (5, 17, 33), (2, 35, 70), (70, 15, 31)])
def test_first_layers_at_tile_edges(channels, pools, n, H, W):
    """The bf16 layers that read the frames (16 x 32 and 8 x 32 tiles; 70 frames: one tile each; (2, 35, 70) and 5 frames of
    17 x 33: ragged ones), alone, as a pair and with the pool, against the oracle's steps with bf16 storage.  Sums taken in
    another order turn single roundings of a stored value: at most 2^-8 of it in each of the two layers behind the first."""
    spec = ClassifierSpec(precision=1, channels=channels, pool_after=pools, taps=(1, 2, 3), n_classes=7)
    c, blob = _clf(spec, 72)
    fr = np.random.RandomState(H * W).randint(0, 256, (n, 3, H, W)).astype(np.uint8)
    for ep in (1, 2, 3):
        log = c.classify_chunk(to_dev(fr), ep, want_logits=True)[2]
        torch.cuda.synchronize()
        some = [0, n - 1]
        ref = oc.classify(blob, fr[some], ep)["logits"]
        assert relerr(log.cpu().numpy()[some], ref) <= 2.0 ** -7, (ep, relerr(log.cpu().numpy()[some], ref))


@pytest.mark.parametrize("channels,pools", [((64, 64, 64), (2,)), ((64, 64, 64), ()), ((64, 64, 64), (1, 2)), ((128, 64, 64), (1,))])
@pytest.mark.parametrize("n,H,W", [(1, 1, 1), (3, 4, 5), (5, 17, 33), (2, 35, 70)])
def test_first_layers_are_the_general_layers_bit_for_bit(channels, pools, n, H, W):
    """Which kernel runs the first layers is not seen in an answer: logits of every exit are those of the convolution kernel
    on the normalised frames (zero channels up to 64), layer by layer, with biases that are not zero."""
    spec = ClassifierSpec(precision=1, channels=channels, pool_after=pools, taps=(1, 2, 3), n_classes=7)
    blob = make_classifier_blob(spec, 73)
    t = split_classifier_blob(spec, blob)
    rs = np.random.RandomState(H * W + len(pools))
    for k in t:
        if k.endswith(".b"):
            t[k][...] = 0.3 * rs.randn(*t[k].shape)
    from paper_2102_08481_amd import thia_classifier_load
    c = thia_classifier_load(blob, spec.n_exits)
    m, _ = gpu_model(MINI_BF16, 0xBEEF + 51)
    fr = rs.randint(0, 256, (n, 3, H, W)).astype(np.uint8)
    x = np.zeros((n, H, W, 64), np.float32)
    x[..., :3] = (nchw_to_nhwc(fr).astype(np.float32) - np.float32(spec.mean)) / np.float32(spec.std)
    x = to_dev(x, torch.bfloat16)
    for i in (1, 2, 3):
        if i > 1 and i - 1 in pools:
            if min(x.shape[1:3]) < 2:
                break                                   # nothing left behind this pool
            x = c.op_pool(x)
        w = t[f"conv{i}.w"]
        if i == 1:
            w = np.concatenate([w, np.zeros((w.shape[0], 61, 3, 3), np.float32)], 1)
        x = m.op_conv(x, w, t[f"conv{i}.b"], pad=1, relu=True)
        ref = c.op_unit(x.reshape(n, -1, x.shape[-1]), i)
        got = c.classify_chunk(to_dev(fr), i, want_logits=True)
        torch.cuda.synchronize()
        assert torch.equal(got[2], ref[2]), (i, float((got[2] - ref[2]).abs().max()))
        assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
    c.close()


def test_first_pair_walks_several_tiles_per_block():
    """More tiles than blocks (60 frames of 3 x 4 tiles on 256 blocks): every frame's answer is that of the frame alone."""
    spec = ClassifierSpec(precision=1, channels=(64, 64, 64), pool_after=(2,), taps=(2, 3), n_classes=7)
    c, _ = _clf(spec, 72)
    fr = to_dev(np.random.RandomState(3).randint(0, 256, (60, 3, 41, 100)).astype(np.uint8))
    for ep in (1, 2):
        log = c.classify_chunk(fr, ep, want_logits=True)[2]
        one = torch.cat([c.classify_chunk(fr[i:i + 1], ep, want_logits=True)[2] for i in (0, 17, 59)])
        torch.cuda.synchronize()
        assert torch.equal(log[[0, 17, 59]], one)
