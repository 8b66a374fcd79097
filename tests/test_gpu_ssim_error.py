"""The loss gradient of strips of columns is no further from float64 than the
plain float32 evaluation with the five moments x, y, x^2, y^2 and xy: noisy
images, smooth ones (whose variances are small differences), nearly equal and
equal ones."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

f32 = np.float32
W, H, LAM = 1110, 730, 0.2


def blur(img, g, fma):
    for axis in (1, 0):
        p = np.pad(img, [(5, 5) if a == axis else (0, 0) for a in range(3)])
        n, acc = img.shape[axis], np.zeros_like(img)
        for k in range(11):
            t = np.take(p, range(k, k + n), axis=axis)
            acc = (t.astype(np.float64) * g[k] + acc).astype(img.dtype) if fma else acc + g[k] * t
        img = acc
    return img


def five_moments(x, y, dtype):
    """L's gradient times the number of values, in float32 (sums of fused
    multiply-adds) or float64."""
    g = np.exp(-np.arange(-5, 6) ** 2 / (2 * 1.5 ** 2))
    g = (g / g.sum()).astype(dtype)
    c1, c2, lam, two = dtype(0.01) ** 2, dtype(0.03) ** 2, dtype(LAM), dtype(2)
    x, y = x.astype(dtype), y.astype(dtype)
    b = lambda a: blur(a, g, dtype is f32)  # noqa: E731
    mx, my = b(x), b(y)
    sxx, syy, sxy = b(x * x) - mx * mx, b(y * y) - my * my, b(x * y) - mx * my
    a1, a2, b1, b2 = two * mx * my + c1, two * sxy + c2, mx * mx + my * my + c1, sxx + syy + c2
    s = (a1 * a2) / (b1 * b2)
    dm = s * (two * my / a1 - two * my / a2 - two * mx / b1 + two * mx / b2)
    ds = b(dm) + two * x * b(-s / b2) + y * b(two * s / a2)
    return (dtype(1) - lam) * np.sign(x - y) - lam * ds


def images(kind):
    rng = np.random.default_rng(len(kind))
    if kind == "noisy":
        y = rng.random((H, W, 3))
        x = np.clip(y + 0.1 * rng.standard_normal(y.shape), 0, 1)
    else:
        v, u = np.mgrid[:H, :W]
        y = np.stack([0.5 + 0.4 * np.sin(u / 20 + c) * np.cos(v / 15) for c in range(3)], axis=2)
        x = y + {"smooth": 0.02, "near": 1e-3, "equal": 0.0}[kind] * rng.standard_normal(y.shape)
    return x.astype(f32), y.astype(f32)


@pytest.mark.parametrize("kind", ["noisy", "smooth", "near", "equal"])
def test_no_further_from_float64(kind):
    from paper_2411_14974_amd.binding import Renderer
    x, y = images(kind)
    R = Renderer(0)
    try:
        g, _ = R.ssim_loss_grad(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), LAM)
        got = g.cpu().numpy().astype(np.float64) * x.size
    finally:
        R.close()
    want = five_moments(x, y, np.float64)
    plain = float(np.linalg.norm(five_moments(x, y, f32) - want))
    mine = float(np.linalg.norm(got - want))
    print(f"[ssim error] {kind}: {mine:.3e}, five moments {plain:.3e}, of {np.linalg.norm(want):.3e}", flush=True)
    assert mine <= plain
