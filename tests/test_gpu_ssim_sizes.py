"""The loss goes through strips of 226 float columns or through 16 x 16 tiles by
the time that either takes for an image's width and height: large images of
widths at the edges of strips (75, 226, 301, 5351: 0.996, 3, 3.996 and 71.03
strips), shallow and narrow ones, against the oracle (float64) to the bars of
the loss (1e-5 relative) and its gradient (1e-3 of the largest element), and a
gradient written over one of the images on either way."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def R():
    from paper_2411_14974_amd.binding import Renderer
    r = Renderer(0)
    yield r
    r.close()


def images(w, h):
    rng = np.random.default_rng(1000 * w + h)
    x = rng.uniform(0, 1, (h, w, 3)).astype(np.float32)
    return x, np.clip(x + rng.normal(0, 0.1, x.shape), 0, 1).astype(np.float32)


@pytest.mark.parametrize("w,h", [(75, 12001), (226, 3600), (301, 2500), (5351, 149), (4000, 200), (1110, 730),  # strips
                                 (76, 9001), (16, 4096), (1, 700), (2403, 302), (17, 31)])                      # tiles
def test_matches_oracle(R, w, h):
    from oracle import losses
    x, y = images(w, h)
    g, loss = R.ssim_loss_grad(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), 0.3)
    want, gref = losses.loss_and_grad(x.astype(np.float64), y.astype(np.float64), 0.3)
    got, gg = float(loss.cpu()[0]), g.cpu().numpy().astype(np.float64)
    err = float(np.abs(gg - gref).max() / np.abs(gref).max())
    print(f"[ssim sizes {w}x{h}] loss {got:.7f} vs {want:.7f}, grad max err / max |g| {err:.1e}", flush=True)
    assert abs(got - want) <= 1e-5 * abs(want)
    assert err <= 1e-3


@pytest.mark.parametrize("over", ["rgb", "target"])
@pytest.mark.parametrize("w,h", [(1200, 640), (300, 200)])
def test_gradient_over_an_image(R, over, w, h):
    x, y = (torch.from_numpy(a).cuda() for a in images(w, h))
    g, loss = R.ssim_loss_grad(x, y)
    t = {"rgb": x.clone(), "target": y.clone()}
    g2, loss2 = R.ssim_loss_grad(t["rgb"], t["target"], grad=t[over])
    assert torch.equal(g, g2) and torch.equal(loss, loss2)
