"""The nearest-neighbour search along the curve (clouds of more than 768
points) against an exhaustive float32 search with the same distance arithmetic:
sizes at the edges of leaves (16 points) and nodes (1024), and clouds that are
hard for it: far outliers, coincident points, one plane, coordinates far from
the origin, values that are not finite."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def R():
    from paper_2411_14974_amd.binding import Renderer
    r = Renderer(0)
    yield r
    r.close()


def exhaustive(xyz):
    """Mean distance to the three nearest other points (0 for a point that is not finite)."""
    n = xyz.shape[0]
    out = torch.empty(n, device=xyz.device)
    for a in range(0, n, 1000):
        q = xyz[a:a + 1000]
        d = xyz[None] - q[:, None]
        d = (d[..., 0] * d[..., 0] + d[..., 1] * d[..., 1]) + d[..., 2] * d[..., 2]
        d = torch.where(d < float("inf"), d, float("inf"))
        d[torch.arange(q.shape[0]), torch.arange(a, a + q.shape[0])] = float("inf")
        s = torch.sort(d, dim=1).values[:, :3]
        m = (s < float("inf")).sum(1)
        t = torch.where(s < float("inf"), s.sqrt(), 0.0)
        out[a:a + 1000] = torch.where(m > 0, ((t[:, 0] + t[:, 1]) + t[:, 2]) / m.clamp_min(1), 0.0)
    return out


@pytest.mark.parametrize("n,form", [(769, "cube"), (1024, "cube"), (1025, "patches"), (4096, "patches"), (4097, "patches"),
                                    (20011, "patches"), (5000, "outliers"), (3000, "coincident"), (6000, "plane"),
                                    (9000, "far"), (2500, "not finite"), (1300, "all coincident"),
                                    (1100, "none finite")])
def test_curve_search_is_exhaustive(R, n, form):
    from paper_2411_14974_amd.binding import make_init_params
    g = torch.Generator(device="cuda").manual_seed(n)
    xyz = torch.rand(n, 3, device="cuda", generator=g)
    if form == "patches":
        c = torch.rand(16, 3, device="cuda", generator=g) * 4
        xyz = c[torch.randint(0, 16, (n,), device="cuda", generator=g)] + xyz * torch.tensor([0.5, 0.3, 0.001], device="cuda")
    elif form == "outliers":
        xyz[:40] = (xyz[:40] - 0.5) * 1e7
    elif form == "coincident":
        xyz[n // 2:] = xyz[:n - n // 2]
    elif form == "plane":
        xyz[:, 1] = 0.25
    elif form == "far":
        xyz += torch.tensor([5e5, -3e5, 100.0], device="cuda")
    elif form == "not finite":
        xyz[::7, 0] = float("nan")
        xyz[3::11, 2] = float("inf")
        xyz[5] = 3e38
    elif form == "all coincident":
        xyz[:] = 0.5
    elif form == "none finite":
        xyz[:] = float("nan")
    # one direction of unit length times the radius, without the centre's rounding: the spread of the points
    ds = R.init_from_points(xyz, None, 6, 0, make_init_params(radius_scale=1.0, radius_min=1e-12))
    ok = torch.isfinite(xyz).all(1)
    want = exhaustive(xyz).clamp_min(1e-12).double()
    got = (ds.points.double() - xyz.double()[:, None]).norm(dim=2).mean(1)
    # a point's coordinates round to half an ulp of their size
    size = xyz.double().abs().amax(1) + want
    err = ((got - want).abs() / (want * 1e-6 + size * 2.0 ** -23))[ok]
    worst = float(err.max()) if err.numel() else 0.0
    print(f"[curve search] n={n} {form}: worst error {worst:.2f} of the rounding bound", flush=True)
    assert worst <= 1.0
    assert torch.isfinite(ds.points[ok]).all()
