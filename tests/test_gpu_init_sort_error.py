"""The neighbour search along the curve does without the sort where that
reports that a wait ran out: the points keep the cloud's order, with the same
distances bit for bit."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [769, 1000, 5003, 20000])
def test_failed_sort_is_not_used(n):
    from paper_2411_14974_amd import binding
    L = binding.lib()
    size = getattr(L, "_ZN2cs23neighbour_scratch_bytesEi")      # cs::neighbour_scratch_bytes(int)
    search = getattr(L, "_ZN2cs22launch_neighbour_meansEP12ihipStream_tiPKfPhj")  # cs::launch_neighbour_means(...)
    size.argtypes, size.restype = [C.c_int], C.c_size_t
    search.argtypes, search.restype = [C.c_void_p, C.c_int, C.c_void_p, C.c_void_p, C.c_uint32], None
    g = torch.Generator(device="cuda").manual_seed(n)
    xyz = torch.randn(n, 3, device="cuda", generator=g) * torch.tensor([1.0, 0.2, 5.0], device="cuda")
    xyz[::9, 1] = float("nan")
    xyz[5:8] = xyz[10]
    xyz[3] = 3e38
    out = []
    for err0 in (0, 1):
        scratch = torch.zeros(size(n), dtype=torch.uint8, device="cuda")
        search(torch.cuda.current_stream().cuda_stream, n, xyz.data_ptr(), scratch.data_ptr(), err0)
        torch.cuda.synchronize()
        out.append(scratch[:4 * n].view(torch.float32).clone())
    assert float(out[0].max()) > 0.0
    assert torch.equal(out[0], out[1])
    print(f"[init sort error] {n} points: same distances", flush=True)
