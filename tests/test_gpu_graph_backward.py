"""Backward passes of captured frames: a backward repeated, and captured before
the forward was, gives the eager gradients at every replay (a captured cell sort
can leave its lists in another buffer than the eager first frame's)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2411_14974_amd import scenes  # noqa: E402


@pytest.fixture(scope="module")
def R():
    from paper_2411_14974_amd.binding import Renderer
    r = Renderer(0)
    yield r
    r.close()


# 1, 2 and 3 passes of the cell sort, eager and captured in turn
@pytest.mark.parametrize("sizes", [((200, 150),), ((1300, 900),), ((700, 500), (640, 400)), ((1920, 1080),),
                                   ((513, 256), (330, 420), (979, 546))])
def test_repeated_backward_of_captured_frames(R, sizes):
    from paper_2411_14974_amd.binding import FLAG_GRAPH, DeviceScene, make_params
    rng = np.random.default_rng(len(sizes) + sizes[0][0])
    sc = scenes.convexes_around(rng, scenes.gmm_centres(rng, 5000), 5, 1)
    cams = [scenes.orbit_camera(rng, w, h) for w, h in sizes]
    ds = DeviceScene.from_scene(sc, "cuda:0")
    dls = [torch.from_numpy(rng.normal(size=(c.height, c.width, 3)).astype(np.float32)).cuda() for c in cams]
    _, st = R.forward_batch(ds, cams, make_params(), want_state=True)
    want = {k: v.double() for k, v in R.backward_batch(st, dls).items()}
    st.release()
    out = {k: torch.empty(v.shape, device="cuda") for k, v in want.items()}
    for _ in range(4):
        _, st = R.forward_batch(ds, cams, make_params(flags=FLAG_GRAPH), want_state=True)
        for _ in range(3):
            for v in out.values():
                v.fill_(float("nan"))
            got = R.backward_batch(st, dls, grads=out)
            torch.cuda.synchronize()
            for k in want:
                # sums of up to some thousand float32 terms in another order
                assert float((got[k].double() - want[k]).norm() / want[k].norm().clamp_min(1e-30)) <= 1e-5, k
        st.release()
