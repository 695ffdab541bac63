"""The head's decode writes the logits of gs_images.n_pixels pixels and no others."""
import numpy as np
import pytest

from paper_2412_01217_amd import scenes
from tests.test_gpu_list_edges import one_tile

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_classes", [13, 52])
@pytest.mark.parametrize("sizes,pixels", [
    ([(20, 20), (24, 12)], 400),          # the first of two items
    ([(20, 20), (24, 12)], 250),          # a part of it, past a multiple of 64
    ([(20, 20), (24, 12)], 500),          # the first and a part of the second
    ([(8, 8), (8, 8), (40, 40)], 64),     # one chunk
    ([(20, 20), (24, 12)], 688),          # all
])
def test_decode_ends_at_n_pixels(sizes, pixels, n_classes):
    from paper_2412_01217_amd import raster
    sc, _ = one_tile(60, 16, True, False, seed=3)
    sc.emb, sc.sem = scenes.f32_to_bf16_bits(sc.sem), None
    views = [scenes.identity_view(W, H, W, W, W / 2, H / 2, 1) for W, H in sizes]
    cfg = raster.config(16)
    fr = raster.Frame(cfg, views)
    g = raster.to_device(sc)
    proj = raster.preprocess(cfg, g, fr)
    srt = raster.bin_sort(cfg, proj, fr, sc.n)
    r = np.random.default_rng(1)
    bits = lambda *s: torch.from_numpy(scenes.f32_to_bf16_bits(r.normal(size=s).astype(np.float32)).view(np.int16)).cuda()  # noqa: E731
    real = lambda *s: torch.from_numpy(r.normal(size=s).astype(np.float32)).cuda()  # noqa: E731
    head = dict(W1=bits(64, 16), b1=real(64), W2=bits(n_classes, 64), b2=real(n_classes))
    full = raster.render_fwd(cfg, g, proj, fr, srt, head=head)["logits"]
    out = raster.alloc_images(cfg, fr, n_classes, True)
    out["n_pixels"] = pixels
    out["logits"].fill_(7.0)              # (the buffer holds all of them)
    got = raster.render_fwd(cfg, g, proj, fr, srt, out=out, head=head)["logits"]
    want = torch.full_like(full, 7.0)
    base = 0
    for W, H in sizes:
        HW, here = W * H, max(0, min(W * H, pixels - base))
        plane = slice(base * n_classes, (base + HW) * n_classes)
        want[plane].view(n_classes, HW)[:, :here] = full[plane].view(n_classes, HW)[:, :here]
        base += HW
    assert torch.equal(got, want)
