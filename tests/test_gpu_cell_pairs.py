"""A convex makes a (cell, convex) pair only of cells in which it keeps a tile:
slanted slivers, whose tile rectangles are mostly empty, have complete lists in
views with cells of one, 2 x 2 and 4 x 4 tiles, and the limits that are stated
in (tile, convex) pairs hold for them (a replayed frame's margin, the
allocation-free forward's scratch)."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from gpu_helpers import NAMES, say  # noqa: E402
from paper_2411_14974_amd import scenes  # noqa: E402


@pytest.fixture(scope="module")
def R():
    from paper_2411_14974_amd.binding import Renderer
    r = Renderer(0)
    yield r
    r.close()


def slivers(rng, n, w, h, length, angle, spread, opacity=0.5):
    """n slivers of `length` pixels at `angle`, some 2 pixels thick, with centres within
    `spread` pixels of the image centre of a w x h view of focal length w."""
    z = rng.uniform(3.0, 5.0, n)
    uv = rng.uniform(-spread, spread, (n, 2))
    along = np.array([math.cos(angle), math.sin(angle)])
    across = np.array([-along[1], along[0]])
    corners = np.array([(-0.5, -1.0), (-0.5, 1.0), (0.0, -1.3), (0.0, 1.3), (0.5, -1.0), (0.5, 1.0)])
    q = uv[:, None, :] + length * corners[None, :, :1] * along + corners[None, :, 1:] * across
    points = np.concatenate([q * (z / w)[:, None, None], np.broadcast_to(z[:, None, None], (n, 6, 1))], axis=2)
    f = lambda a: np.ascontiguousarray(a, np.float32)  # noqa: E731
    return scenes.Scene(f(points), np.full(n, 50.0, np.float32), np.full(n, 20.0, np.float32), np.full(n, opacity, np.float32),
                        f(rng.uniform(-1.0, 1.0, (n, 1, 3))))


def front(w, h, roll=0.0, zoom=1.0):
    c, s = math.cos(roll), math.sin(roll)
    return scenes.Camera(w, h, w * zoom, w * zoom, w / 2.0, h / 2.0, np.array([[c, -s, 0], [s, c, 0], [0, 0, 1]]))


def rectangle_tiles(R, ds, cam):
    rects = np.array([d.tile_rect[:] for d in R.debug_preprocess(ds, cam)], np.int64)
    sides = np.maximum(rects[:, 2:] - rects[:, :2] + 1, 0)
    return int((sides[:, 0] * sides[:, 1]).sum())


@pytest.mark.parametrize("tile,w,h,length", [
    (16, 512, 256, 90), (16, 512, 256, 400),      # cells of one tile; rectangles of up to 64 tiles, larger ones
    (16, 513, 300, 110), (16, 700, 500, 600),     # cells of 2 x 2
    (8, 700, 500, 60), (8, 700, 500, 700),        # cells of 4 x 4
])
@pytest.mark.parametrize("angle", [0.05, 0.6, 2.2])
def test_lists_of_slivers(R, tile, w, h, length, angle):
    import oracle
    from paper_2411_14974_amd.binding import DeviceScene, make_params
    rng = np.random.default_rng(w + length)
    sc = slivers(rng, 400, w, h, length, angle, min(w, h) / 3)
    cam = front(w, h)
    ds = DeviceScene.from_scene(sc, "cuda:0")
    rgb, st = R.forward(ds, cam, make_params(tile=tile), want_state=True)
    ranges, ids = st.tile_lists()
    pairs = st.stats()["pairs"]
    st.release()
    assert pairs == int((ranges[:, 1] - ranges[:, 0]).sum())
    keys = np.array([c.key for c in oracle.preprocess(sc, cam)], np.uint64)
    tx_n = (w + tile - 1) // tile
    for t in rng.choice(ranges.shape[0], 40, replace=False):
        lst = ids[ranges[t, 0]:ranges[t, 1]]
        assert len(set(lst.tolist())) == len(lst)
        assert np.all(np.lexsort((lst, keys[lst])) == np.arange(len(lst))), t
        cand = oracle.tile_candidates(sc, cam, tile, int(t % tx_n), int(t // tx_n))
        assert set(cand.tolist()) <= set(lst.tolist()), t
    ref, _, _ = oracle.render(sc, cam, mode=oracle.MODE_MATCHED)
    assert float(np.abs(rgb.cpu().numpy().astype(np.float64) - ref).max()) <= 1e-4
    say(f"[slivers] tile {tile}, {w}x{h}, length {length}, angle {angle}: {pairs} pairs")


def test_replay_within_the_margin_is_accepted(R):
    """Slivers seen level, then slanted: their tile pairs stay within the replayed
    frame's 30 %, the tiles of their rectangles do not."""
    from paper_2411_14974_amd.binding import FLAG_GRAPH, DeviceScene, make_params
    rng = np.random.default_rng(8)
    sc = slivers(rng, 3000, 512, 256, 90, 0.0, 60)
    ds = DeviceScene.from_scene(sc, "cuda:0")
    level, slanted = front(512, 256, zoom=1.5), front(512, 256, roll=math.pi / 4)
    dl = [torch.from_numpy(rng.normal(size=(256, 512, 3)).astype(np.float32)).cuda()]
    pairs = []
    for cam in (level, slanted):
        ref, s = R.forward_batch(ds, [cam], make_params(), want_state=True)
        want = R.backward_batch(s, dl)
        pairs.append(s.stats()["pairs"])
        s.release()
    rect = rectangle_tiles(R, ds, slanted)
    say(f"[slivers] level {pairs[0]}, slanted {pairs[1]} tile pairs, {rect} tiles of rectangles")
    assert pairs[1] <= 1.3 * pairs[0] < rect
    for cam in (level, level, slanted):
        out, st = R.forward_batch(ds, [cam], make_params(flags=FLAG_GRAPH), want_state=True)
        assert R.batch_check(st) == 0
        g = R.backward_batch(st, dl)
        torch.cuda.synchronize()
        st.release()
    assert torch.equal(out[0], ref[0])
    for k in NAMES:
        assert float((g[k].double() - want[k].double()).norm() / want[k].double().norm().clamp_min(1e-30)) <= 1e-5, k


def test_allocation_free_forward_within_its_limit(R):
    """100k slivers whose rectangles hold more tiles than the scratch has room for
    pairs, and whose kept tiles fit."""
    from paper_2411_14974_amd.binding import DeviceScene, make_params
    rng = np.random.default_rng(9)
    sc = slivers(rng, 100_000, 512, 256, 520, math.atan2(1, 2), 20)
    ds = DeviceScene.from_scene(sc, "cuda:0")
    cam = front(512, 256)
    ref, st = R.forward(ds, cam, make_params(), want_state=True)
    pairs, rect = st.stats()["pairs"], rectangle_tiles(R, ds, cam)
    st.release()
    say(f"[slivers] {pairs} tile pairs, {rect} tiles of rectangles")
    assert 17 * pairs < (480 << 20) and 16 * rect > (512 << 20)
    out = torch.full_like(ref, float("nan"))
    R.forward_noalloc(ds, cam, out)
    assert torch.equal(out, ref)
