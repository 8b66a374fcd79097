"""The SSIM loss kernel walks strips of 226 float columns (75.3 pixels) down
segments of rows: images at the edges of strips and segments and smaller than
the 11-pixel window, against the oracle (float64) to the bars of the loss
(1e-5 relative) and its gradient (1e-3 of the largest element), and a gradient
written over one of the images."""
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


@pytest.mark.parametrize("w,h", [(1, 1), (1, 40), (5, 3), (75, 11), (76, 12), (151, 64), (226, 21), (640, 1), (333, 410), (1000, 530), (1031, 653)])
def test_matches_oracle(R, w, h):
    from oracle import losses
    x, y = images(w, h)
    g, loss = R.ssim_loss_grad(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), 0.3)
    want, gref = losses.loss_and_grad(x.astype(np.float64), y.astype(np.float64), 0.3)
    got, gg = float(loss.cpu()[0]), g.cpu().numpy().astype(np.float64)
    err = float(np.abs(gg - gref).max() / np.abs(gref).max())
    print(f"[ssim strips {w}x{h}] loss {got:.7f} vs {want:.7f}, grad max err / max |g| {err:.1e}", flush=True)
    assert abs(got - want) <= 1e-5 * abs(want)
    assert err <= 1e-3


@pytest.mark.parametrize("over", ["rgb", "target"])
def test_gradient_over_an_image(R, over):
    x, y = (torch.from_numpy(a).cuda() for a in images(300, 170))
    g, loss = R.ssim_loss_grad(x, y)
    t = {"rgb": x.clone(), "target": y.clone()}
    g2, loss2 = R.ssim_loss_grad(t["rgb"], t["target"], grad=t[over])
    assert torch.equal(g, g2) and torch.equal(loss, loss2)
