"""Binning by cell: a cell of 1, 2 x 2 or 4 x 4 tiles holds one list, and a
tile's list is the cell's filtered by the tile's mask bit.  At sizes on both
sides of every rule (512 cells a view; cells of 4 x 4 at most; more than 65 536
cells in a call, which changes the key layout), with ragged edges, every tile's
list holds the oracle's candidates in depth order, and images and gradients do
not depend on the binning."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from gpu_helpers import say  # noqa: E402
from paper_2411_14974_amd import scenes  # noqa: E402


@pytest.fixture(scope="module")
def R():
    from paper_2411_14974_amd.binding import Renderer
    r = Renderer(0)
    yield r
    r.close()


def a_scene(n, w, h, seed):
    rng = np.random.default_rng(seed)
    sc = scenes.convexes_around(rng, scenes.uniform_centres(rng, n), 6, 0)
    return sc, scenes.orbit_camera(rng, w, h)


# (tile, width, height): tiles across x down -> cells
@pytest.mark.parametrize("tile,w,h", [
    (16, 5, 3),        # 1 tile
    (16, 512, 256),    # 32 x 16 = 512 tiles: cells of one tile
    (16, 513, 256),    # 33 x 16 = 528 tiles: cells of 2 x 2, a ragged column
    (8, 360, 360),     # 45 x 45 tiles -> 23 x 23 = 529 cells of 2 x 2: cells of 4 x 4, ragged both ways
    (32, 1920, 1080),  # 60 x 34 -> 30 x 17 = 510 cells of 2 x 2
    (8, 700, 500),     # 88 x 63 tiles, 4 x 4
])
def test_lists_hold_candidates_in_order(R, tile, w, h):
    import oracle
    from paper_2411_14974_amd.binding import DeviceScene, make_params
    sc, cam = a_scene(700, w, h, w + h)
    ds = DeviceScene.from_scene(sc, "cuda:0")
    rgb, st = R.forward(ds, cam, make_params(tile=tile), want_state=True)
    ranges, ids = st.tile_lists()
    keys = np.array([c.key for c in oracle.preprocess(sc, cam)], np.uint64)
    tx_n = (w + tile - 1) // tile
    assert ranges.shape[0] == tx_n * ((h + tile - 1) // tile)
    assert st.stats()["pairs"] == int((ranges[:, 1] - ranges[:, 0]).sum()) == len(ids)
    rng = np.random.default_rng(1)
    some = rng.choice(ranges.shape[0], min(40, ranges.shape[0]), replace=False)
    for t in some:
        lst = ids[ranges[t, 0]:ranges[t, 1]]
        assert len(set(lst.tolist())) == len(lst)
        assert np.all(np.lexsort((lst, keys[lst])) == np.arange(len(lst))), t
        cand = oracle.tile_candidates(sc, cam, tile, int(t % tx_n), int(t // tx_n))
        assert set(cand.tolist()) <= set(lst.tolist()), t
    st.release()
    say(f"[cells] tile {tile}, {w}x{h}: {len(some)} lists hold their candidates in depth order, {len(ids)} pairs")


def test_long_lists_and_sparse_hits(R):
    """Tiles whose lists pass many rounds of the list reader, with convexes far
    smaller than a tile (few of a cell's entries are a given tile's) and faint
    enough that no pixel is ever done: the image equals the oracle's, the
    gradients those of the 8-pixel and 32-pixel tilings."""
    import oracle
    from paper_2411_14974_amd.binding import DeviceScene, make_params
    rng = np.random.default_rng(11)
    n = 30000
    sc = scenes.convexes_around(rng, scenes.uniform_centres(rng, n, (-0.9,) * 3, (0.9,) * 3), 6, 0)
    c = sc.points.mean(axis=1, keepdims=True)
    sc.points = np.ascontiguousarray(c + 0.08 * (sc.points - c), np.float32)
    sc.opacity = np.full(n, 0.02, np.float32)
    sc.sigma, sc.delta = np.full(n, 20.0, np.float32), np.full(n, 50.0, np.float32)
    cam = scenes.orbit_camera(rng, 150, 110)
    ds = DeviceScene.from_scene(sc, "cuda:0")
    ref, _, _ = oracle.render(sc, cam)
    dl = torch.from_numpy(rng.normal(size=(110, 150, 3)).astype(np.float32)).cuda()
    grads = {}
    for tile in (8, 16, 32):
        rgb, st = R.forward(ds, cam, make_params(tile=tile), want_state=True)
        grads[tile] = R.backward(st, dl)
        ranges, _ = st.tile_lists()
        err = float(np.abs(rgb.cpu().numpy().astype(np.float64) - ref).max())
        say(f"[long lists] tile {tile}: longest list {int((ranges[:, 1] - ranges[:, 0]).max())}, "
            f"image max |gpu - oracle| {err:.2e}")
        st.release()
        assert err <= 1e-4
    for k, g in grads[16].items():
        for tile in (8, 32):
            gap = float((grads[tile][k].double() - g.double()).norm() / g.double().norm().clamp_min(1e-30))
            assert gap <= 1e-5, (k, tile, gap)


def test_more_cells_than_16_bits(R):
    """8200 x 8200 pixels in tiles of 8: more than 65 536 cells of 4 x 4, so the
    keys hold 28 bits of cell (2 x 2 tiles); the image equals the 32-pixel
    tiling's bit for bit."""
    from paper_2411_14974_amd.binding import DeviceScene, make_params
    sc, cam = a_scene(200, 8200, 8200, 3)
    ds = DeviceScene.from_scene(sc, "cuda:0")
    a, _ = R.forward(ds, cam, make_params(tile=8))
    b, _ = R.forward(ds, cam, make_params(tile=32))
    assert float(a.abs().max()) > 0.0
    assert torch.equal(a, b)
    say("[cells] 28-bit cell keys: image equals the 32-pixel tiling's")


def test_batch_of_views_with_different_cells(R):
    """Views of one call with cells of 1, 2 x 2 and 4 x 4 tiles: images equal
    the views rendered alone."""
    from paper_2411_14974_amd.binding import DeviceScene, make_params
    sc, _ = a_scene(5000, 64, 64, 9)
    rng = np.random.default_rng(4)
    cams = [scenes.orbit_camera(rng, w, h) for w, h in ((64, 48), (640, 360), (1297, 840), (17, 9))]
    ds = DeviceScene.from_scene(sc, "cuda:0")
    outs, st = R.forward_batch(ds, cams, make_params(), want_state=True)
    torch.cuda.synchronize()
    for c, o in zip(cams, outs):
        alone, _ = R.forward(ds, c, make_params())
        assert torch.equal(alone, o)
    st.release()


@pytest.mark.parametrize("k", [3, 4, 5, 6, 7, 8])
def test_small_views_split_by_record(R, k):
    """Small views are composited by squares with the records split over the
    wavefronts, a call with many pixels by tiles: the same scene seen alone and
    in a batch with a large view gives the same images bit for bit, the same
    work counts, and gradients equal up to the order of their sums."""
    from paper_2411_14974_amd.binding import DeviceScene, make_params
    rng = np.random.default_rng(70 + k)
    sc = scenes.convexes_around(rng, scenes.uniform_centres(rng, 4000), k, 1)
    cams = [scenes.orbit_camera(rng, w, h) for w, h in ((1000, 700), (61, 83), (8, 8), (250, 130))]
    ds = DeviceScene.from_scene(sc, "cuda:0")
    p = make_params(background=(0.2, 0.4, 0.6))
    dls = [torch.from_numpy(rng.normal(size=(c.height, c.width, 3)).astype(np.float32)).cuda() for c in cams]
    outs, st = R.forward_batch(ds, cams, p, want_state=True)
    g = R.backward_batch(st, dls)
    both = st.counters()
    st.release()
    total, alone = {n: 0.0 for n in g}, {n: 0 for n in both}
    for c, o, dl in zip(cams, outs, dls):
        img, s1 = R.forward(ds, c, p, want_state=True)
        g1 = R.backward(s1, dl)
        cnt = s1.counters()
        s1.release()
        assert torch.equal(img, o), (k, c.width)
        for n in total:
            total[n] = total[n] + g1[n].double()
        for n in alone:
            alone[n] += cnt[n]
    for n in g:
        gap = float((total[n] - g[n].double()).norm() / total[n].norm().clamp_min(1e-30))
        assert gap <= 1e-5, (k, n, gap)
    # (a batch's pairs and tests depend on nothing but the views; the record's
    # evaluations counted per wavefront alike)
    for n in ("pairs", "tested", "full", "full_bwd", "sum_T_full", "wave_evals"):
        assert alone[n] == both[n], (k, n, alone[n], both[n])
