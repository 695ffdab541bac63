"""Compositing and its reverse pass at the edges of their batches: tile lists of 1 to 330 entries
(the kernels take 64 list entries at a time, 32 or 16 Gaussians per matrix-core batch and 8x8
pixel regions), channel counts around the padded widths, and feature arrays whose rows cannot
be read as vectors."""
import numpy as np
import pytest

import oracle
from paper_2412_01217_amd import scenes
from tests.helpers import check_with_pixel_terms, flagged, pixel_mask_to_channels, rel_check

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

FWD_TOL = 1e-4    # the bars of the other parity tests
BWD_TOL = 1e-3


def one_tile(n, n_sem, faint, compact, seed=0):
    """n Gaussians on one 16x16 tile (every rectangle meets it): faint (no pixel is ever full) or
    opaque (most pixels stop), compact (a few pixels each, most miss a given region) or wide."""
    rng = np.random.default_rng(9000 + 7 * n + n_sem + seed)
    z = rng.uniform(2.0, 4.0, n)
    u, v = rng.uniform(0.5, 15.5, n), rng.uniform(0.5, 15.5, n)
    mean = np.stack([(u - 8) / 16 * z, (v - 8) / 16 * z, z], 1)
    q = rng.normal(size=(n, 4))
    sc = scenes.Scene(mean.astype(np.float32), rng.normal(-2.6 if compact else -1.0, 0.4, (n, 3)).astype(np.float32),
                      (q / np.linalg.norm(q, axis=1, keepdims=True)).astype(np.float32),
                      rng.normal(-3.5 if faint else 1.0, 0.3, n).astype(np.float32),
                      rng.uniform(0, 1, (n, 3)).astype(np.float32), rng.normal(size=(n, n_sem)).astype(np.float32), None,
                      n_sem)
    return sc, [scenes.identity_view(16, 16, 16.0, 16.0, 8.0, 8.0, 1)]


def render(sc, views, n_sem, state, g=None, **kw):
    from paper_2412_01217_amd import raster
    cfg = raster.config(n_sem, **kw)
    fr = raster.Frame(cfg, views)
    g = raster.to_device(sc) if g is None else g
    if n_sem == 0:
        g.pop("sem", None)
    proj = raster.preprocess(cfg, g, fr)
    srt = raster.bin_sort(cfg, proj, fr, sc.n)
    img = raster.render_fwd(cfg, g, proj, fr, srt, split=state)
    return raster, cfg, fr, g, proj, srt, img


LENGTHS = [1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 95, 96, 97, 128, 129, 330]


@pytest.mark.parametrize("faint,compact", [(True, False), (True, True), (False, True)])
@pytest.mark.parametrize("n", LENGTHS)
@pytest.mark.parametrize("n_sem,state", [(5, True), (29, False)])
def test_list_lengths(n, n_sem, state, faint, compact):
    check(n, n_sem, state, faint, compact)


@pytest.mark.parametrize("n_sem", [0, 1, 2, 3, 4, 6, 7, 12, 20, 22, 23, 27, 28, 29, 32, 52, 54, 55, 59, 60])
def test_channel_counts(n_sem):
    check(75, n_sem, True, True, True)


def check(n, n_sem, state, faint, compact):
    sc, views = one_tile(n, n_sem, faint, compact)
    raster, cfg, fr, g, proj, srt, img = render(sc, views, n_sem, state)
    K = 4 + n_sem
    ocfg = oracle.Config()
    ref = oracle.render(ocfg, sc, views)
    flag = flagged(ref["flag"], f"n={n}", bound=0.05)
    its = oracle.items(views)
    mask = pixel_mask_to_channels(flag, its, K)
    # sum of the terms' magnitudes: the render of |features|
    asc = sc.copy()
    asc.rgb, asc.sem = np.abs(sc.rgb), np.abs(sc.sem)
    scale = oracle.render(ocfg, asc, views)["img"]
    rel_check(img["color"].cpu().numpy(), ref["img"], FWD_TOL, mask=mask, scale=scale, name="color")
    rel_check(img["T"].cpu().numpy(), ref["T"], FWD_TOL, mask=flag, name="T")
    assert (img["n_contrib"].cpu().numpy()[~flag] == ref["n_contrib"].reshape(-1)[~flag]).all()
    gimg = np.random.default_rng(n).normal(size=256 * K).astype(np.float32)
    gimg[mask] = 0.0
    gin = dict(color=torch.from_numpy(gimg).cuda(), logits=None)
    grads = raster.render_bwd(cfg, g, proj, fr, srt, img, gin)
    gref = oracle.backward(ocfg, sc, views, gimg)
    gabs = oracle.backward(ocfg, sc, views, np.abs(gimg))
    pre = None
    for f in ("rgb", "sem") if n_sem else ("rgb",):
        rel_check(grads[f].cpu().numpy(), gref[f], BWD_TOL, scale=gabs[f], name=f)
    for f in ("mean", "log_scale", "quat", "opacity"):
        pre = check_with_pixel_terms(grads[f].cpu().numpy(), gref[f], BWD_TOL, f, ocfg, sc, views, gimg, K, pre=pre)


def shifted(t):
    """The same values one element past a 16-byte boundary."""
    base = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
    out = base[1:].view(t.shape)
    out.copy_(t)
    return out


@pytest.mark.parametrize("learned,n_sem", [(False, 20), (False, 52), (True, 16)])
def test_rows_that_are_no_vectors(learned, n_sem):
    """A feature array that starts off a 16-byte boundary is read value by value: same image and
    the same gradients up to the order of the atomic sums."""
    sc, views = one_tile(150, n_sem, False, True)
    if learned:
        sc.emb, sc.sem = scenes.f32_to_bf16_bits(sc.sem), None
    out = []
    for move in (False, True):
        from paper_2412_01217_amd import raster
        g = raster.to_device(sc)
        key = "emb" if learned else "sem"
        if move:
            g[key] = shifted(g[key])
            assert g[key].data_ptr() % 16 != 0
        r, cfg, fr, g, proj, srt, img = render(sc, views, n_sem, True, g=g)
        gin = dict(color=torch.linspace(-1, 1, img["color"].numel(), device="cuda"), logits=None)
        out.append((img, r.render_bwd(cfg, g, proj, fr, srt, img, gin, grads=r.alloc_grads(cfg, g, fr, 16))))
    (a, ga), (b, gb) = out
    assert torch.equal(a["color"], b["color"]) and torch.equal(a["n_contrib"], b["n_contrib"])
    for k in ("mean", "opacity", "rgb", "emb" if learned else "sem"):
        d = (ga[k] - gb[k]).abs().max().item()
        assert d <= 1e-5 * ga[k].abs().max().item(), (k, d)
