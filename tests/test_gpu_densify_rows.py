"""Split and prune copy rows in accesses as wide as the row length and the
arrays' alignment allow: for every K and SH degree, at sizes round a block of
256, with aligned and unaligned input arrays, decisions and copies are the
oracle's bit for bit."""
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


def shifted(t):  # the same values one element past an aligned address
    buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
    buf[1:].copy_(t.reshape(-1))
    return buf[1:].view(t.shape)


@pytest.mark.parametrize("unaligned", [(), ("points",), ("sh",)])
@pytest.mark.parametrize("n,k,deg", [(1, 3, 0), (255, 4, 1), (256, 5, 2), (257, 6, 3), (700, 7, 0), (513, 8, 1), (300, 6, 2),
                                     (1000, 4, 3)])
def test_rows_match_oracle(R, n, k, deg, unaligned):
    from oracle import densify as D
    from paper_2411_14974_amd.binding import DeviceScene, make_densify_params
    rng = np.random.default_rng(n * k + deg)
    sc = scenes.convexes_around(rng, scenes.uniform_centres(rng, n), k, deg)
    sc.opacity[rng.random(n) < 0.2] = 0.01
    denom = rng.integers(0, 4, n).astype(np.float32)
    accum = (np.where(rng.random(n) < 0.3, rng.uniform(5e-6, 1e-4, n), rng.uniform(0, 3e-6, n)) * denom).astype(np.float32)
    p = make_densify_params()
    ds = DeviceScene.from_scene(sc, "cuda:0")
    for name in unaligned:
        setattr(ds, name, shifted(getattr(ds, name)))
    out, src = R.densify(ds, torch.from_numpy(accum).cuda(), torch.from_numpy(denom).cuda(), p)
    torch.cuda.synchronize()
    pts, dl, sg, op, sh, rsrc = D.densify(sc, accum, denom, p.opacity_min, p.size_max, p.split_threshold, p.child_scale,
                                          p.child_sigma_scale, p.child_opacity_scale)
    assert np.array_equal(src.cpu().numpy(), rsrc)
    for got, want in ((out.delta, dl), (out.sigma, sg), (out.opacity, op), (out.sh, sh)):
        assert np.array_equal(got.cpu().numpy(), want.astype(np.float32))
    # children: a few float32 roundings of coordinates of about 1; kept rows are copies
    kept = rsrc.shape[0] - k * int(np.sum(np.unique(rsrc, return_counts=True)[1] == k))
    got = out.points.cpu().numpy()
    assert np.array_equal(got[:kept], sc.points[rsrc[:kept]].reshape(kept, k, 3))
    assert float(np.abs(got.astype(np.float64) - pts).max(initial=0.0)) <= 2e-6
