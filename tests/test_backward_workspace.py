"""The reverse pass's workspace may start anywhere: its double-precision records are aligned inside
it, and the size that gs_workspace_size asks for has room for that. An aligned one needs no more."""
import ctypes
import os

import numpy as np
import pytest

from paper_2412_01217_amd import _lib as L


def required(items=2, n=10, tiles=4, cap=0):
    c = L.Config()
    L.lib().gs_config_default(ctypes.byref(c))
    b = ctypes.c_size_t()
    assert L.lib().gs_workspace_size(L.GS_WS_RENDER_BWD, ctypes.byref(c), items, n, tiles, cap, 0, ctypes.byref(b)) == 0
    return b.value


def call(address, ws_bytes):
    """gs_render_bwd with placeholder pointers (never dereferenced on the host)."""
    c = L.Config()
    L.lib().gs_config_default(ctypes.byref(c))
    fake = ctypes.c_void_p(256)
    g = L.Gaussians(10, fake, fake, fake, fake, fake, None, None)
    p = L.Projected(fake, fake, fake)
    im = L.Images(fake, fake, fake, None, 100, None, 0)
    gr = L.Grads(*([fake] * 12))
    return L.lib().gs_render_bwd(ctypes.byref(c), ctypes.byref(g), ctypes.byref(p), fake, 1, fake, 2, 4, fake, fake, None,
                                 ctypes.byref(im), ctypes.byref(im), ctypes.byref(gr), ctypes.c_void_p(address), ws_bytes,
                                 None)


@pytest.mark.skipif(os.path.exists("/dev/kfd"), reason="host-only check: placeholder pointers must never reach a GPU")
def test_size_covers_the_alignment():
    """Without a GPU a call whose arguments are good comes back with GS_ERR_HIP, from its first launch."""
    full = required()
    for address in (4096, 4097, 4098, 4100, 4104, 4108, 4111):
        skip = -address % 16
        assert call(address, full) == L.GS_ERR_HIP, address
        assert call(address, full - 16 + skip) == L.GS_ERR_HIP, address
        assert call(address, full - 16 + skip - 1) == L.GS_ERR_WORKSPACE, address


@pytest.mark.gpu
@pytest.mark.parametrize("offset", [1, 4, 8, 12])
def test_workspace_off_its_boundary(offset):
    torch = pytest.importorskip("torch")
    from paper_2412_01217_amd import raster, scenes
    from tests.test_gpu_list_edges import one_tile, render
    sc, _ = one_tile(330, 5, True, False, seed=9)
    views = [scenes.identity_view(40, 24, 30.0, 30.0, levels=2)]
    _, cfg, fr, g, proj, srt, img = render(sc, views, 5, True, seg_len=256)
    gin = dict(color=torch.linspace(-1, 1, img["color"].numel(), device="cuda"), logits=None)
    size = raster.workspace_bytes(L.GS_WS_RENDER_BWD, cfg, fr, sc.n, srt.capacity)
    out = []
    for skip in (0, offset):
        whole = torch.full((size + 32,), 0xA5, dtype=torch.uint8, device="cuda")
        assert whole.data_ptr() % 16 == 0
        grads = raster.render_bwd(cfg, g, proj, fr, srt, img, gin, ws=whole[skip:skip + size])
        assert (whole[:skip] == 0xA5).all() and (whole[skip + size:] == 0xA5).all()
        out.append({k: v.cpu().numpy() for k, v in grads.items() if v is not None})
    for k in ("mean", "log_scale", "quat", "opacity", "rgb", "sem", "pose"):
        a, b = (o[k].astype(np.float64) for o in out)
        # the same sums in another order of their atomics
        assert np.abs(a - b).max() <= 1e-5 * np.abs(a).max(), k
