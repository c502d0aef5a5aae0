"""Designs whose cells crowd into a few bands of the density scatter (early in a
placement), against the FP64 oracle: relative L2 <= 1e-5, the bar of every float32
result here.  The library's sums do not depend on the order of its lists, so the
calls that share them agree bit for bit."""
import dataclasses

import numpy as np
import pytest

import gen
import oracle
from _helpers import rel_l2
from gpu_common import RTOL, DeviceCells, host, lib_or_build, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    lib_or_build()
    from paper_1312_4587_amd import fftpl
    return fftpl


# lists of a band as the counting blocks of 512 cells leave them: `each` cells of
# every block in the lowest rows and the rest above, at the lengths where a list's
# owner is written in another way (32, 33), empty lists among them, and all cells in
# one band (many windows of entries)
@pytest.mark.parametrize("m,n,each,skip", [(8193, 256, 32, 1), (9000, 256, 33, 1),
                                           (20000, 512, 31, 3), (20001, 512, 34, 3),
                                           (20000, 512, 512, 1), (60000, 64, 200, 2),
                                           (300001, 1024, 4096, 1),
                                           (16384, 256, 300, 1), (16385, 256, 300, 1),
                                           (8192, 257, 512, 1), (8193, 512, 400, 1),
                                           (8192, 1, 512, 1), (100000, 16, 512, 2)])
def test_density_of_crowded_bands(F, m, n, each, skip):
    import torch
    inst = gen.make_instance((110, m, n, each), num_cells=m, util=0.7, n=n, num_nets=1)
    i = np.arange(m)
    low = (i % 512 < each) & (i // 512 % skip == 0)
    rng = np.random.default_rng((111, m))
    rows = np.where(low, rng.uniform(0.6, 1.4, m), rng.uniform(8, max(9, n - 2), m))
    inst = dataclasses.replace(inst, y=(inst.yl + rows * inst.bin_h).astype(np.float32))
    c, grid = DeviceCells(inst), F.Grid.of(inst)
    a, b = (torch.full((n * n,), 5.0, device="cuda") for _ in range(2))
    say("crowded density", m, n, each, skip)
    F.density_map(grid, c.x, c.y, c.w, c.h, None, a)
    F.problem_density(F.Problem.from_instance(inst), c.x, c.y, b)
    torch.cuda.synchronize()
    zero = np.zeros((n, n))
    assert rel_l2(host(a).reshape(n, n), oracle.density_map(inst, zero)) < RTOL
    assert torch.equal(a, b)   # (the problem's fixed map is zero)


# one workspace for the map alone (bands of single rows on grids of up to 256) and
# for evaluations (row pairs), in turn
@pytest.mark.parametrize("m,n,dct", [(20000, 256, "fft"), (70000, 8, "fft"),
                                     (9000, 192, "gemm_f32"), (30000, 320, "gemm_f32")])
def test_map_and_evaluation_share_a_workspace(F, m, n, dct):
    import torch
    inst = gen.make_instance((112, m, n), num_cells=m, util=0.7, n=n, num_nets=m)
    plan, prob, c = F.Plan(n, dct), F.Problem.from_instance(inst), DeviceCells(inst)
    rho = torch.empty(n * n, device="cuda")
    want = oracle.evaluate(inst, lam=1.5, grad_mode="field")
    runs = []
    for _ in range(2):
        say("map, then evaluation", m, n)
        F.problem_density(prob, c.x, c.y, rho)
        gx, gy = (torch.empty(m, device="cuda") for _ in range(2))
        out = torch.empty(4, dtype=torch.float64, device="cuda")
        F.eval(plan, prob, c.x, c.y, 1.5, inst.gamma, "field", gx, gy, out)
        torch.cuda.synchronize()
        assert rel_l2(host(rho).reshape(n, n), want["rho"]) < RTOL
        assert torch.equal(plan.maps()[0].reshape(-1), rho)
        runs.append((gx, gy, out))
    assert all(torch.equal(a, b) for a, b in zip(*runs))
    assert rel_l2(host(runs[0][0]), want["gx"]) < RTOL
    assert rel_l2(host(runs[0][1]), want["gy"]) < RTOL
    plan.close()
