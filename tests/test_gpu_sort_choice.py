"""Which method the automatic choice of gs_bin_sort takes. The radix path leaves the same bytes in its
workspace every time it sorts the same entries, and the bucket path others."""
import numpy as np
import pytest

from paper_2412_01217_amd import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def workspace(sort_mode, views, n, radius, capacity):
    from paper_2412_01217_amd import raster
    cfg = raster.config(0, sort_mode=sort_mode)
    fr = raster.Frame(cfg, views)
    rng = np.random.default_rng(n)
    E = fr.n_items * n
    rec = np.zeros((E, 8), np.float32)
    rec[:, :2] = rng.uniform(1, 15, (E, 2))
    proj = dict(rec=torch.from_numpy(rec.reshape(-1)).cuda(),
                depth=torch.from_numpy(rng.uniform(1, 9, E).astype(np.float32)).cuda(),
                radius=torch.full((E,), radius, dtype=torch.int32, device="cuda"))
    s = raster.Sorter(cfg, fr, n, capacity)
    s.ws.fill_(0xA5)
    s.run(proj)
    assert int(s.status.item()) == 0
    return s.ws


LINE = {1: 2560, 2: 2048}   # entries and capacity a tile


@pytest.mark.parametrize("items,tiles", [(1, 5), (2, 5)])
@pytest.mark.parametrize("n,capacity,radix", [
    ("over", "over", True),        # both pass the line
    ("over", "at", False),         # the capacity, sized to a frame that meets few tiles, does not
    ("at", "over", False),         # the entries do not
    ("few", "over", False),        # no list can pass 8192 keys
])
def test_automatic_choice(items, tiles, n, capacity, radix):
    """Every rectangle meets the first tile of its item only."""
    line = LINE[items] * tiles * items
    count = {"over": line // items + 1, "at": line // items, "few": 8192}[n]
    views = [scenes.identity_view(16 * tiles, 16, levels=1)] * items
    if n == "few":
        views = [scenes.identity_view(16, 16, levels=1)] * items
        line = LINE[items] * items
    cap = max(line, items * count) + 1 if capacity == "over" else line
    radius = 1
    if capacity == "at" and items * count > cap:
        cap, radius = line, 0      # (as many duplicates as fit: none)
    ws = [workspace(m, views, count, radius, cap) for m in (0, 1)]
    assert torch.equal(*ws) == radix
