"""Calls with more (cell, convex) pairs than a call can hold are refused, also
where a 32-bit sum of the counts comes out small: convexes that fill 16384 x
16384 pixels in tiles of 8 make 2^20 pairs each, so 4096 of them 2^32."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from gpu_helpers import say  # noqa: E402
from paper_2411_14974_amd import scenes  # noqa: E402

SIDE = 16384


def square(side):
    return scenes.Camera(side, side, float(side), float(side), side / 2.0, side / 2.0)


def triangles(n, size):
    """n triangles round the optical axis at depths 2 to 3, `size` times their depth wide."""
    z = np.linspace(2.0, 3.0, n)
    c = np.array([(-1.0, -1.0), (1.0, -1.0), (0.0, 1.5)]) * size
    p = np.concatenate([c[None] * z[:, None, None], np.broadcast_to(z[:, None, None], (n, 3, 1))], axis=2)
    f = lambda v: np.full(n, v, np.float32)  # noqa: E731
    return scenes.Scene(np.ascontiguousarray(p, np.float32), f(2.0), f(2.0), f(0.5), np.full((n, 1, 3), 0.5, np.float32))


# one workgroup orders the first, one tile of the pair scan is full of the second
@pytest.mark.parametrize("n", [4096, 163 * 4096])
def test_wrapped_sums_are_refused(n):
    from paper_2411_14974_amd.binding import CS_ENOMEM, CSError, DeviceScene, Renderer, make_params
    R = Renderer(0)
    try:
        cam = square(SIDE)
        out = torch.empty((SIDE, SIDE, 3), device="cuda:0")
        p = make_params(tile=8)
        filled = DeviceScene.from_scene(triangles(n, 100.0), "cuda:0")
        some = [d.tile_rect[:] for d in R.debug_preprocess(DeviceScene.from_scene(triangles(4, 100.0), "cuda:0"), cam, p)]
        assert some == [[0, 0, SIDE // 8 - 1, SIDE // 8 - 1]] * 4
        for reused in (False, True):  # a new frame, then one that holds pair buffers
            if reused:
                R.forward(DeviceScene.from_scene(triangles(n, 1e-4), "cuda:0"), cam, p, out=out)
            with pytest.raises(CSError) as e:
                R.forward(filled, cam, p, out=out)
            assert e.value.code == CS_ENOMEM
            say(f"[pair limit] {n} convexes over {SIDE}^2, {'reused' if reused else 'new'} frame: {e.value}")
    finally:
        R.close()


def test_tile_pairs_saturate():
    """4096 convexes over 8192 x 8192 pixels in tiles of 8: 2^28 cell pairs, which a
    call can hold, that stand for 2^32 tile pairs."""
    from paper_2411_14974_amd.binding import DeviceScene, Renderer, make_params
    R = Renderer(0)
    try:
        cam, p = square(8192), make_params(tile=8)
        ds = DeviceScene.from_scene(triangles(4096, 100.0), "cuda:0")
        out, st = R.forward(ds, cam, p, want_state=True)
        assert st.counters()["pairs"] == (1 << 32) - 1
        st.release()
        few, _ = R.forward(DeviceScene.from_scene(triangles(4096, 100.0).subset(np.arange(64)), "cuda:0"), cam, p)
        assert torch.equal(few, out)  # (what lies behind the first 64 is never seen)
    finally:
        R.close()
