"""Results of blocking calls come through host memory that a pool shared by all
threads hands out: 24 threads (more than the pool keeps pieces for), each with
its own stream, arrays and radii, get the results that they get one by one."""
from concurrent.futures import ThreadPoolExecutor

import pytest

from gpu_helpers import announce, torch_cuda

pytestmark = pytest.mark.gpu


def test_threads_get_their_own_results():
    announce("24 threads: projections and iterations at once")
    torch = torch_cuda()
    import paper_2510_00562_amd as geo
    jobs = []
    for q in range(24):
        g = torch.Generator(device="cuda").manual_seed(q)
        v = 0.5 + 0.1 * torch.randn((5, 20 + q, 33), generator=g, device="cuda")
        p = geo.params(0.3, 4.0 + q, 2.0, omega=0.03)
        d = geo.dims_of(v.shape)
        jobs.append((v, p, d, geo.Workspace(geo.geo_workspace_size(d, p)), torch.cuda.Stream()))
    torch.cuda.synchronize()

    def run(job):
        v, p, d, ws, stream = job
        n, st, out = v.numel(), stream, []
        with torch.cuda.stream(stream):
            buf = torch.empty(n, device="cuda")
        geo.geo_state_init(d, p, v, ws, stream=st)
        for k in range(5):
            out.append(geo.geo_project_l1(v.view(-1), 0.1 * (k + 1) * n, buf, stream=st))
            out.append(geo.geo_project_l2(v.view(-1), buf, 0.01, buf, stream=st))
            r = geo.geo_step(d, p, v, ws, 3, stream=st)
            out += [r.total_iters, r.tau_s, r.tau_t, r.r, r.rel_change]
        return out

    alone = [run(j) for j in jobs]
    assert len({tuple(a) for a in alone}) == len(jobs)
    with ThreadPoolExecutor(24) as pool:
        assert list(pool.map(run, jobs)) == alone
