"""View-dependent features and their backward where the kernels' groups end: 16 Gaussians a wave,
16 channels a load, four views at a time; every pair of degrees; directions that do not exist."""
import numpy as np
import pytest

from oracle import sh as osh
from paper_2412_01217_amd import scenes
from tests.helpers import rel_check

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-5   # of the sum of the terms' sizes: single precision, up to 60 channels x 15 bands x 5 views


def setup(n, S, V, dr, ds, seed=0):
    from paper_2412_01217_amd import raster
    rng = np.random.default_rng(seed + 7 * n + S)
    base = scenes.room_scene(n=64, n_classes=1, seed=5, log_mu=-3.3)
    views = [scenes.identity_view(32, 32, 30.0, 30.0, levels=1)]
    if V > 1:
        views += list(scenes.room_views(base, V - 1, 32, 32, levels=1, seed=9))
    f = lambda *s: rng.normal(size=s).astype(np.float32)   # noqa: E731
    mean = f(n, 3) + np.array([0, 0, 6], np.float32)
    a = dict(mean=mean, rgb=f(n, 3), sem=f(n, S), rr=f(n, osh.n_coeffs(dr) - 1, 3), rs=f(n, osh.n_coeffs(ds) - 1, S),
             gr=f(V, n, 3), gs=f(V, n, S))
    return raster, views, a


def run(raster, views, a, dr, ds, mean0=None):
    n, S, V = len(a["mean"]), a["sem"].shape[1], len(views)
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()   # noqa: E731
    fr = raster.Frame(raster.config(S, view_features=1), views)
    z = lambda *s: torch.zeros(*s, device="cuda")   # noqa: E731
    g = dict(mean=t(a["mean"]), log_scale=z(n, 3), quat=z(n, 4), opacity=z(n), rgb=t(a["rgb"]), sem=t(a["sem"]) if S else None)
    sh = dict(rgb_degree=dr, sem_degree=ds, rgb_rest=t(a["rr"]) if dr else None, sem_rest=t(a["rs"]) if ds and S else None)
    out = raster.sh_features(g, sh, fr)
    grads = dict(rgb=t(a["gr"].reshape(V * n, 3)), sem=t(a["gs"].reshape(V * n, S)) if S else None,
                 mean=t(mean0) if mean0 is not None else z(n, 3), pose=z(V, 6))
    band = raster.sh_features_bwd(g, sh, fr, grads)
    torch.cuda.synchronize()
    c = lambda x: None if x is None else x.cpu().numpy()   # noqa: E731
    return {k: c(v) for k, v in out.items()}, {k: c(v) for k, v in grads.items()}, {k: c(v) for k, v in band.items()}


def check(views, a, dr, ds, out, grads, band, mean0=0.0, keep=slice(None)):
    S, V = a["sem"].shape[1], len(views)
    gm, gp, mm, mp = mean0, 0.0, np.abs(mean0) + 1e-6, 1e-6
    for name, dc, rest, deg, g in (("rgb", a["rgb"], a["rr"], dr, a["gr"]), ("sem", a["sem"], a["rs"], ds, a["gs"])):
        if name == "sem" and S == 0:
            continue
        ref = osh.features(views, a["mean"], dc, rest, deg)
        size = np.abs(dc)[None] + (np.abs(rest).sum(1)[None] if deg else 0)
        rel_check(out[name].reshape(ref.shape)[:, keep], ref[:, keep], TOL, name=name,
                  scale=np.broadcast_to(size, ref.shape)[:, keep])
        gdc, grest, m, p = osh.features_backward(views, a["mean"], rest, deg, g)
        size = np.abs(g).sum(0)
        rel_check(band[name + "_dc"], gdc, TOL, name=name + " constant band", scale=size)
        if deg:
            rel_check(band[name + "_rest"][keep], grest[keep], TOL, name=name + " bands",
                      scale=np.broadcast_to(size[:, None], grest.shape)[keep])
        gm, gp = gm + m, gp + p
        for v, view in enumerate(views):   # |dY/dd| <= 8 up to degree 3
            r = np.maximum(np.linalg.norm(a["mean"] - osh.camera_centre(view), axis=1), 1e-3)
            t = 8.0 * (np.abs(g[v])[:, None] * (np.abs(rest) if deg else 0.0 * np.abs(g[v])[:, None])).sum((1, 2)) / r
            mm = mm + t[:, None]
            mp = mp + np.eye(V)[v][:, None] * t[keep].sum()
    if dr or (ds and S):
        rel_check(grads["mean"][keep], gm[keep], TOL, name="mean", scale=np.broadcast_to(mm, gm.shape)[keep])
        return gp, np.broadcast_to(mp, gp.shape)
    return None, None


CASES = [(n, S, V, dr, ds) for dr in range(4) for ds in range(4)
         for n, S, V in [(37, 20, 2)]] + [(n, S, V, 3, 1) for n, S, V in
                                          [(1, 1, 1), (15, 0, 3), (16, 15, 4), (17, 16, 5), (65, 17, 8), (1000, 52, 2),
                                           (64, 60, 9), (30000, 3, 1)]] + [(33, 33, 5, 0, 3), (129, 60, 3, 2, 2), (50, 8, 2, 1, 2), (35, 16, 1, 3, 3),
                                                      (21, 32, 6, 0, 2)]


@pytest.mark.parametrize("n,S,V,dr,ds", CASES)
def test_matches_oracle(n, S, V, dr, ds):
    raster, views, a = setup(n, S, V, dr, ds)
    mean0 = np.random.default_rng(1).normal(size=(n, 3)).astype(np.float32)
    out, grads, band = run(raster, views, a, dr, ds, mean0)
    gp, mp = check(views, a, dr, ds, out, grads, band, mean0=mean0)
    if gp is not None:
        rel_check(grads["pose"], gp, TOL, name="pose", scale=mp)


@pytest.mark.parametrize("dr,ds", [(3, 1), (0, 2), (1, 0)])
def test_no_gradient_no_share(dr, ds):
    """A Gaussian in the camera's own place, and one with an infinite coefficient: without a
    gradient in that view (that channel) they change nothing; with one, only their own rows."""
    raster, views, a = setup(40, 20, 2, dr, ds, seed=3)
    a["mean"][5] = 0.0                       # the first view's centre
    a["gr"][0, 5] = a["gs"][0, 5] = 0.0
    keep = np.arange(40) != 5
    out, grads, band = run(raster, views, a, dr, ds)
    b = {k: v.copy() for k, v in a.items()}
    b["mean"][5] = 1e-3                      # (a direction for the oracle; its first view has no share)
    gp, mp = check(views, b, dr, ds, out, grads, band, keep=keep)
    for x in [grads["mean"], grads["pose"]] + [v for v in band.values() if v is not None]:
        assert np.isfinite(x).all()
    a["gr"][0, 5, 1] = a["gs"][0, 5, 2] = 1.0
    _, grads, _ = run(raster, views, a, dr, ds)
    assert np.isnan(grads["mean"][5]).all() and np.isfinite(grads["mean"][keep]).all()

    raster, views, a = setup(40, 20, 2, dr, ds, seed=4)
    if dr:
        a["rr"][7, 1, 2], a["gr"][:, 7, 2] = np.inf, 0.0
    if ds:
        a["rs"][9, 2, 19], a["gs"][:, 9, 19] = np.inf, 0.0
    _, grads, band = run(raster, views, a, dr, ds)
    for x in [grads["mean"], grads["pose"]] + [v for v in band.values() if v is not None]:
        assert np.isfinite(x).all()
