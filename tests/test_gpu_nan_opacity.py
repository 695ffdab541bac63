"""A Gaussian with a NaN opacity among ordinary ones: no pixel takes it, so the image and every
other gradient, the poses' included, are those of the scene without it, and of its own gradients
only the opacity's is NaN."""
import numpy as np
import pytest

from paper_2412_01217_amd import scenes
from tests.test_gpu_list_edges import one_tile

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

FIELDS = ("mean", "log_scale", "quat", "opacity", "rgb", "sem", "emb")
TOL = 1e-4


def run(sc, n_sem, state, seg_len):
    """Two views of one tile: image, gradients of a fixed image gradient."""
    from paper_2412_01217_amd import raster
    views = [scenes.identity_view(16, 16, 16.0, 16.0, 8.0, 8.0, 1), scenes.identity_view(16, 16, 16.0, 16.0, 7.0, 9.0, 1)]
    cfg = raster.config(n_sem, seg_len=seg_len)
    fr = raster.Frame(cfg, views)
    g = raster.to_device(sc)
    proj = raster.preprocess(cfg, g, fr)
    srt = raster.bin_sort(cfg, proj, fr, sc.n)
    img = raster.render_fwd(cfg, g, proj, fr, srt, split=state)
    gin = dict(color=torch.linspace(-1, 1, img["color"].numel(), device="cuda"), logits=None)
    grads = raster.render_bwd(cfg, g, proj, fr, srt, img, gin, grads=raster.alloc_grads(cfg, g, fr, 16))
    out = {k: grads[k].cpu().numpy().astype(np.float64) for k in FIELDS + ("pose",) if grads.get(k) is not None}
    return proj["radius"].view(2, sc.n).cpu().numpy(), img, out


# (long lists: split into segments, with the forward's state or with the reverse pass's own summary)
@pytest.mark.parametrize("n,seg_len", [(40, 0), (330, 256)])
@pytest.mark.parametrize("state", [True, False])
@pytest.mark.parametrize("learned,n_sem", [(False, 3), (False, 20), (False, 52), (True, 16)])
def test_nan_opacity_stays_with_its_gaussian(learned, n_sem, state, n, seg_len):
    sc, _ = one_tile(n, n_sem, True, False, seed=5)
    if learned:
        sc.emb, sc.sem = scenes.f32_to_bf16_bits(sc.sem), None
    bad = n // 2
    sc.opacity[bad] = np.nan
    rest = sc.copy()
    for f in FIELDS:
        if getattr(sc, f, None) is not None:
            setattr(rest, f, np.delete(getattr(sc, f), bad, axis=0))
    radius, img, got = run(sc, n_sem, state, seg_len)
    _, iref, ref = run(rest, n_sem, state, seg_len)
    assert (radius[:, bad] > 0).all()
    # single-precision sums of the same terms in another grouping, a pixel's transmittance walked over
    # segments of 256 that end elsewhere (256 steps of 2^-23 are 3e-5): 1e-4 of the largest entry
    for k in ("color", "T"):
        d = (img[k] - iref[k]).abs().max().item()
        assert d <= TOL * iref[k].abs().max().item(), (k, d)
    for k in FIELDS:
        if k not in got:
            continue
        own, others = got[k][bad], np.delete(got[k], bad, axis=0)
        if k == "opacity":
            assert np.isnan(own)
        else:
            assert (own == 0).all(), (k, own)
        assert np.abs(others - ref[k]).max() <= TOL * np.abs(ref[k]).max(), k
    # the pose sums the camera-space means' gradients and their moments (depths and offsets are
    # below 4) over the Gaussians: the same share of the magnitudes that are added up
    scale = 4 * (np.abs(ref["mean"]).sum() + np.abs(ref["log_scale"]).sum())
    assert np.isfinite(got["pose"]).all()
    assert np.abs(got["pose"] - ref["pose"]).max() <= TOL * scale
