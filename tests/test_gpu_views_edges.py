"""The projection's backward over more views than its pose sums are held for at a time (64), and over
more pyramid levels than are read ahead (4): the views of one frame against each view in a frame of
its own. Their terms are the same; sums over blocks, and of the single runs, round to single
precision (2^-24 of each part)."""
import numpy as np
import pytest

from paper_2412_01217_amd import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def gradients(g, views, seed):
    from paper_2412_01217_amd import raster
    cfg = raster.config(4)
    fr = raster.Frame(cfg, views)
    n = g["mean"].shape[0]
    proj = raster.preprocess(cfg, g, fr)
    srt = raster.bin_sort(cfg, proj, fr, n)
    img = raster.render_fwd(cfg, g, proj, fr, srt)
    gin = torch.cat([torch.from_numpy(np.random.default_rng(seed + k).normal(size=sum(
        (v.W >> l) * (v.H >> l) for l in range(v.levels)) * 8).astype(np.float32)) for k, v in enumerate(views)]).cuda()
    out = raster.render_bwd(cfg, g, proj, fr, srt, img, dict(color=gin, logits=None))
    return {k: out[k].cpu().numpy().astype(np.float64) for k in ("mean", "log_scale", "quat", "opacity", "pose")}


@pytest.mark.parametrize("n_views,side,levels", [(1, 32, 6), (3, 32, 5), (63, 16, 1), (64, 16, 1), (65, 16, 2), (130, 16, 1)])
def test_views_together_and_alone(n_views, side, levels):
    from paper_2412_01217_amd import raster
    sc = scenes.room_scene(n=600, n_classes=4, seed=31, log_mu=-2.5)
    views = scenes.room_views(sc, n_views, side, side, fx=side / 2, levels=levels, seed=8)
    g = raster.to_device(sc)
    got = gradients(g, views, 50)
    one = [gradients(g, [v], 50 + k) for k, v in enumerate(views)]
    pose = np.concatenate([o["pose"] for o in one])
    assert np.abs(pose).max(1).min() > 0.0
    # three blocks' parts of a view, each rounded once; parts may be larger than their sum
    np.testing.assert_allclose(got["pose"], pose, rtol=0, atol=1e-5 * np.abs(pose).max())
    for k in ("mean", "log_scale", "quat", "opacity"):
        ref, size = sum(o[k] for o in one), sum(np.abs(o[k]) for o in one)
        assert (np.abs(got[k] - ref) <= 2.0 ** -22 * size + 1e-12).all(), k
