"""A captured frame with more pairs than its buffers were sized for stays
reported, at every check and backward, until the next forward, which makes room
for it: views of more than 512 tiles, whose cell pairs fit where their tile
pairs do not, and small ones, where neither do."""
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


@pytest.mark.parametrize("w,h", [(256, 160), (640, 400), (1297, 840)])
def test_overflow_is_reported_until_the_next_forward(R, w, h):
    from paper_2411_14974_amd.binding import (CS_EOVERFLOW, FLAG_GRAPH, CSError, DeviceScene, make_camera, make_params)
    rng = np.random.default_rng(w)
    sc = scenes.convexes_around(rng, scenes.uniform_centres(rng, 6000), 6, 1)
    cams = [scenes.orbit_camera(rng, w, h) for _ in range(2)]
    far = [make_camera(c) for c in cams]
    for c in far:  # from further away: far fewer pairs
        c.t[2] = c.t[2] + 8.0
    ds = DeviceScene.from_scene(sc, "cuda:0")
    graph, eager = make_params(flags=FLAG_GRAPH), make_params()
    dls = [torch.from_numpy(rng.normal(size=(h, w, 3)).astype(np.float32)).cuda() for _ in cams]
    ref, s = R.forward_batch(ds, cams, eager, want_state=True)
    gref = R.backward_batch(s, dls)
    pairs = s.stats()["pairs"]
    s.release()
    for first in (far, far):  # sized, then captured
        _, st = R.forward_batch(ds, first, graph, want_state=True)
        assert R.batch_check(st) == 0
        assert 1.3 * st.stats()["pairs"] < pairs
        st.release()
    _, st = R.forward_batch(ds, cams, graph, want_state=True)
    for _ in range(2):
        assert R.batch_check(st) == CS_EOVERFLOW
    for _ in range(2):
        with pytest.raises(CSError) as e:
            R.backward_batch(st, dls)
        assert e.value.code == CS_EOVERFLOW
    assert R.batch_check(st) == CS_EOVERFLOW
    st.release()
    for _ in range(3):
        outs, st = R.forward_batch(ds, cams, graph, want_state=True)
        assert R.batch_check(st) == 0
        g = R.backward_batch(st, dls)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(outs, ref))
        for k in NAMES:
            assert float((g[k].double() - gref[k].double()).norm() / gref[k].double().norm()) <= 1e-5, k
        st.release()
    say(f"[overflow {w}x{h}] reported until the next forward, which makes room for {pairs} pairs")


def test_state_of_a_replaced_frame_is_refused(R):
    """A state whose frame was given up for another scene's is refused, also where
    the new frame lies at the old one's address."""
    from paper_2411_14974_amd.binding import CS_EINVAL, FLAG_GRAPH, CSError, DeviceScene, make_params
    rng = np.random.default_rng(3)
    cams = [scenes.orbit_camera(rng, 200, 150)]
    dls = [torch.from_numpy(rng.normal(size=(150, 200, 3)).astype(np.float32)).cuda()]
    p = make_params(flags=FLAG_GRAPH)
    held = []
    for _ in range(4):
        ds = DeviceScene.from_scene(scenes.convexes_around(rng, scenes.uniform_centres(rng, 3000), 6, 1), "cuda:0")
        _, st = R.forward_batch(ds, cams, p, want_state=True)
        for old in held:
            assert R.batch_check(old) == CS_EINVAL
            with pytest.raises(CSError) as e:
                R.backward_batch(old, dls)
            assert e.value.code == CS_EINVAL
        assert R.batch_check(st) == 0
        held.append(st)
    for st in held:
        st.release()
