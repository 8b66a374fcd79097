"""Captured frames replayed with other resolutions: calls of few pixels are
composited by record, of many by tile, each by a graph of its own, whichever is
captured first; images, gradients and work counts are the eager call's."""
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


LARGE, SMALL = ((640, 400), (333, 250)), ((200, 150), (61, 83))


@pytest.mark.parametrize("k", [4, 6])
@pytest.mark.parametrize("order", ["LSLSSL", "LLSLS"])
def test_replays_of_large_and_small_views(R, k, order):
    from paper_2411_14974_amd.binding import FLAG_GRAPH, DeviceScene, make_params
    rng = np.random.default_rng(k)
    sc = scenes.convexes_around(rng, scenes.uniform_centres(rng, 4000), k, 1)
    ds = DeviceScene.from_scene(sc, "cuda:0")
    cams = {n: [scenes.orbit_camera(rng, w, h) for w, h in sizes] for n, sizes in (("L", LARGE), ("S", SMALL))}
    dls = {n: [torch.from_numpy(rng.normal(size=(c.height, c.width, 3)).astype(np.float32)).cuda() for c in cs]
           for n, cs in cams.items()}
    want = {}
    for n in cams:
        outs, st = R.forward_batch(ds, cams[n], make_params(), want_state=True)
        want[n] = outs, R.backward_batch(st, dls[n]), st.counters()
        st.release()
    grads = {n: torch.empty_like(getattr(ds, n)) for n in NAMES}
    for step, n in enumerate(order):
        outs, st = R.forward_batch(ds, cams[n], make_params(flags=FLAG_GRAPH), want_state=True)
        for again in range(2):  # the graphs without and with their clearing pass
            R.backward_batch(st, dls[n], grads=grads)
            torch.cuda.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(outs, want[n][0])), (step, n)
            for g in NAMES:
                ref = want[n][1][g].double()
                assert float((grads[g].double() - ref).norm() / ref.norm().clamp_min(1e-30)) <= 1e-5, (step, n, again, g)
            assert st.counters() == want[n][2], (step, n, again)
        assert R.batch_check(st) == 0
        st.release()
    say(f"[graph sizes] K = {k}, {order}: replays equal the eager calls")
