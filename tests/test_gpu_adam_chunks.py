"""The Adam step updates every array in chunks of 1024 elements, 16 bytes at a
time where the arrays are aligned for it: at sizes round a chunk and round 4
elements, with aligned and unaligned arrays, the result is the float64 formula's
to float32 rounding and does not depend on the alignment or on the activated
output."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

NAMES = ("points", "delta", "sigma", "opacity", "sh")


@pytest.fixture(scope="module")
def R():
    from paper_2411_14974_amd.binding import Renderer
    r = Renderer(0)
    yield r
    r.close()


# n * 3k and n * 3(deg + 1)^2 elements: below 4, round 1024 and 2048, several chunks; rows of 3 to 48
@pytest.mark.parametrize("n,k,deg", [(1, 3, 0), (3, 5, 1), (113, 6, 2), (114, 6, 3), (2048, 4, 3), (2049, 3, 0), (4099, 7, 1)])
@pytest.mark.parametrize("offset", [0, 1, 2])
def test_chunks_match_float64(R, n, k, deg, offset):
    from paper_2411_14974_amd.binding import make_adam_params
    nc = (deg + 1) ** 2
    shapes = {"points": (n, k, 3), "delta": (n,), "sigma": (n,), "opacity": (n,), "sh": (n, nc, 3)}
    rng = np.random.default_rng(n)
    draw = lambda scale: {q: (scale * rng.normal(size=s)).astype(np.float32) for q, s in shapes.items()}  # noqa: E731
    raw0, m0, g0 = draw(1.0), draw(0.1), draw(0.1)
    v0 = {q: np.abs(x) for q, x in draw(0.01).items()}

    def put(x):  # `offset` elements past an aligned address
        buf = torch.zeros(x.size + offset, dtype=torch.float32, device="cuda")
        t = buf[offset:].view(x.shape)
        t.copy_(torch.from_numpy(x))
        return t
    lr = dict(lr_points=1e-3, lr_delta=0.005, lr_sigma=0.0045, lr_opacity=0.05, lr_sh_dc=0.0025, lr_sh_rest=1e-4)
    rates = {q: np.full(s, lr.get("lr_" + q, 0.0)) for q, s in shapes.items()}
    rates["sh"][:, :1], rates["sh"][:, 1:] = lr["lr_sh_dc"], lr["lr_sh_rest"]
    got = []
    for with_act in (True, False):
        raw, m, v = ({q: put(x) for q, x in d.items()} for d in (raw0, m0, v0))
        act = {q: put(np.zeros(s, np.float32)) for q, s in shapes.items()} if with_act else None
        R.adam_step({q: put(x) for q, x in g0.items()}, raw, m, v, act, make_adam_params(5, eps=1e-8, **lr))
        torch.cuda.synchronize()
        got.append({q: (raw[q].cpu().numpy(), m[q].cpu().numpy(), v[q].cpu().numpy()) for q in NAMES})
        if act:
            a = {q: act[q].cpu().numpy().astype(np.float64) for q in NAMES}
    b1, b2 = 0.9, 0.999
    for q in NAMES:
        r, g, m, v = (d[q].astype(np.float64) for d in (raw0, g0, m0, v0))
        s = 1 / (1 + np.exp(-r))
        g = g * (np.exp(r) if q in ("delta", "sigma") else s * (1 - s) if q == "opacity" else 1.0)
        m, v = b1 * m + (1 - b1) * g, b2 * v + (1 - b2) * g * g
        new = r - rates[q] / (1 - b1 ** 5) * m / (np.sqrt(v) / np.sqrt(1 - b2 ** 5) + 1e-8)
        fin = np.exp(new) if q in ("delta", "sigma") else 1 / (1 + np.exp(-new)) if q == "opacity" else new
        for have, want in zip((*got[0][q], a[q]), (new, m, v, fin)):
            # a few float32 roundings of values up to about 5
            assert np.all(np.abs(have - want) <= 4e-6 * (np.abs(want) + 1.0)), q
        for x, y in zip(got[0][q], got[1][q]):
            assert np.array_equal(x, y), q
