"""The learned head's decode and its fused loss where 64-pixel chunks end: images of a few
pixels, ragged pyramids, class counts around the 32-class blocks."""
import numpy as np
import pytest

from paper_2412_01217_amd import scenes
from tests.helpers import rel_check, targets_from_random

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# operands are split into two bfloat16 parts, what is left of a product term is below 2^-16 of it
TOL = 2.0 ** -15

VIEWS = {
    "one_pixel": [(1, 1, 1)],
    "63_and_65": [(9, 7, 1), (13, 5, 1)],
    "ragged_pyramid": [(44, 28, 3), (8, 8, 1)],
    "many_chunks": [(200, 136, 3)],
    "all_waves": [(320, 240, 1)],   # more chunks than four waves on every compute unit
}


def setup(views, C, seed=3):
    from paper_2412_01217_amd import raster
    rng = np.random.default_rng(seed + C)
    vs = [scenes.identity_view(W, H, 20.0, 20.0, levels=L) for W, H, L in views]
    cfg = raster.config(16)
    fr = raster.Frame(cfg, vs)
    w = dict(W1=(rng.normal(size=(64, 16)) / 4).astype(np.float32), W2=(rng.normal(size=(C, 64)) / 8).astype(np.float32),
             b1=rng.normal(size=64).astype(np.float32), b2=rng.normal(size=C).astype(np.float32))
    for k in ("W1", "W2"):
        w[k] = scenes.f32_to_bf16_bits(w[k])
    head = {k: torch.from_numpy(v.view(np.int16) if v.dtype == np.uint16 else v).cuda() for k, v in w.items()}
    w64 = {k: (scenes.bf16_bits_to_f32(v) if v.dtype == np.uint16 else v).astype(np.float64) for k, v in w.items()}
    return raster, cfg, fr, vs, head, w64, rng


def planes(fr, img, K):
    for it in fr.item_list():
        HW, pb = it["W"] * it["H"], it["pixel_base"]
        yield it, img[pb * K: pb * K + K * HW].reshape(K, HW)


@pytest.mark.parametrize("C", [1, 13, 31, 32, 33, 52, 64])
@pytest.mark.parametrize("case", list(VIEWS))
def test_decode(case, C):
    raster, cfg, fr, vs, head, w, rng = setup(VIEWS[case], C)
    n = 300
    sc = scenes.tiny_scene(n=n, n_classes=1, seed=11)
    sc.emb = scenes.f32_to_bf16_bits(rng.normal(size=(n, 16)).astype(np.float32))
    sc.sem = None
    g = raster.to_device(sc)
    proj = raster.preprocess(cfg, g, fr)
    srt = raster.bin_sort(cfg, proj, fr, n)
    img = raster.render_fwd(cfg, g, proj, fr, srt, head=head)
    color, logits = img["color"].cpu().numpy().astype(np.float64), img["logits"].cpu().numpy()
    for (it, E), (_, got) in zip(planes(fr, color, 20), planes(fr, logits, C)):
        h = np.maximum(w["W1"] @ E[4:] + w["b1"][:, None], 0.0)
        ref = w["W2"] @ h + w["b2"][:, None]
        mag = np.abs(w["W2"]) @ (np.abs(w["W1"]) @ np.abs(E[4:]) + np.abs(w["b1"])[:, None]) + np.abs(w["b2"])[:, None]
        rel_check(got, ref, TOL, scale=mag, floor=0.0, name=f"logits {it['W']}x{it['H']}")


@pytest.mark.parametrize("C", [1, 31, 33, 52, 64])
@pytest.mark.parametrize("case", list(VIEWS))
def test_fused_loss(case, C):
    """Loss parts, dL/dE and the head's weight gradients of a given embedding image against 64 bits.
    A pixel with a hidden unit near its ReLU's kink is left unlabelled."""
    raster, cfg, fr, vs, head, w, rng = setup(VIEWS[case], C)
    P = fr.n_pixels
    color = rng.normal(size=20 * P).astype(np.float32)
    rgb, depth, lab = targets_from_random(vs, C, invalid_frac=0.2)
    lab = lab.astype(np.int32)
    for it, E in planes(fr, color.astype(np.float64), 20):
        pre = w["W1"] @ E[4:] + w["b1"][:, None]
        near = (np.abs(pre) < 1e-4 * (np.abs(w["W1"]) @ np.abs(E[4:]) + np.abs(w["b1"])[:, None])).any(0)
        lab[it["pixel_base"]: it["pixel_base"] + near.size][near] = -1
    tgt = dict(rgb=torch.from_numpy(rgb).cuda(), depth=torch.from_numpy(depth).cuda(), label=torch.from_numpy(lab).cuda())
    img = dict(color=torch.from_numpy(color).cuda(), T=None, n_contrib=None, logits=None, n_pixels=P)
    grads = {"head_" + k: torch.empty(v.shape, device="cuda") for k, v in w.items()}
    parts, gout = raster.loss(cfg, fr, C, img, tgt, head=head, grads=grads)
    parts, gcol = parts.cpu().numpy(), gout["color"].cpu().numpy()
    W1, W2 = w["W1"], w["W2"]
    gw = {k: np.zeros_like(v) for k, v in w.items()}
    mw = {k: np.zeros_like(v) for k, v in w.items()}
    for i, ((it, E), (_, G)) in enumerate(zip(planes(fr, color.astype(np.float64), 20), planes(fr, gcol, 20))):
        pb, HW = it["pixel_base"], it["W"] * it["H"]
        pre = W1 @ E[4:] + w["b1"][:, None]
        h = np.maximum(pre, 0.0)
        z = W2 @ h + w["b2"][:, None]
        z -= z.max(0)
        p = np.exp(z) / np.exp(z).sum(0)
        y = lab[pb: pb + HW]
        ok = (y >= 0) & (y < C)
        one = np.zeros_like(p)
        one[np.where(ok, y, 0), np.arange(HW)] = ok
        dl = np.where(ok, p - one, 0.0) / HW
        ce = -(np.log(p[np.where(ok, y, 0), np.arange(HW)]) * ok).sum() / HW
        d = E[3] - depth[pb: pb + HW]
        valid = depth[pb: pb + HW] > 0
        ref = [np.abs(E[:3] - rgb[3 * pb: 3 * pb + 3 * HW].reshape(3, HW)).mean(),
               np.abs(d[valid]).sum() / max(valid.sum(), 1), ce]
        np.testing.assert_allclose(parts[i], ref, rtol=1e-4, atol=1e-6)
        dh = (W2.T @ dl) * (pre > 0)
        mh = (np.abs(W2.T) @ np.abs(dl)) * (pre > 0)
        rel_check(G[4:], W1.T @ dh, 1e-3, scale=np.abs(W1.T) @ mh, floor=0.0, name="dE")
        rel_check(G[:3], np.sign(E[:3] - rgb[3 * pb: 3 * pb + 3 * HW].reshape(3, HW)) / (3 * HW), 1e-5, name="drgb")
        for k, x, m in (("W1", dh @ E[4:].T, mh @ np.abs(E[4:]).T), ("b1", dh.sum(1), mh.sum(1)),
                        ("W2", dl @ h.T, np.abs(dl) @ h.T), ("b2", dl.sum(1), np.abs(dl).sum(1))):
            gw[k] += x
            mw[k] += m
    for k in gw:
        rel_check(grads["head_" + k].cpu().numpy(), gw[k], 1e-3, scale=mw[k], floor=0.0, name=k)
