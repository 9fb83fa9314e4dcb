"""A blocking call that fails after its kernels were launched: they write their
results to host memory that later calls of any thread are given, so the call ends
only when its stream has. The failure is an error that another call of the thread
left behind (a device number that does not exist) and that the launch reports."""
import pytest

from gpu_helpers import announce, torch_cuda

pytestmark = pytest.mark.gpu


def test_a_failed_call_waits_for_its_kernels():
    torch = torch_cuda()
    import paper_2510_00562_amd as geo
    announce("a projection that fails on a busy stream")
    n = 1000
    x = torch.linspace(-1.0, 1.0, n, device="cuda")
    out, zero = torch.empty_like(x), torch.zeros_like(x)
    a = torch.ones((4096, 4096), device="cuda")
    stream = torch.cuda.Stream()
    ws = geo.Workspace(1 << 20)
    want = geo.geo_project_l2(x, zero, 0.5, out, ws, stream=stream)
    set_device = geo.lib()["hipSetDevice"]
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        for _ in range(100):
            torch.mm(a, a)
    assert not stream.query()
    assert set_device(9999) != 0
    with pytest.raises(geo.GeoError):
        geo.geo_project_l2(x, zero, 0.5, out, ws, stream=stream)
    assert stream.query()
    assert geo.geo_project_l2(x, zero, 0.5, out, ws, stream=stream) == want
