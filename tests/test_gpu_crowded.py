"""Designs that load the lanes and blocks of a kernel unevenly, against the FP64
oracle (relative L2 <= 1e-5, the bar of every float32 result here): cells crowded
into a few bands of the density scatter, as early in a placement, large cells among
small ones, many cells on small grids, and many pins on few cells.  The library's sums do not depend on the order of its lists, so the
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


# large cells among small ones in the gather that reads one map after the other: a
# wavefront shares out the bins of each (past eight columns or three rows), several to
# a wavefront, none, partly and wholly outside the region
@pytest.mark.parametrize("m,n,share,run", [(524288, 1024, 0.01, 1), (524301, 1030, 0.0001, 1),
                                           (524299, 1024, 0.01, 64)])
def test_field_gather_of_large_cells(F, m, n, share, run):
    import torch
    inst = gen.make_instance((113, m, n), num_cells=m, util=0.7, n=n, num_nets=0)
    rng = np.random.default_rng((114, m))
    # unit bins and dyadic edges, so that float32 and the oracle see the same bins
    big = np.repeat(rng.random(m // run + 1) < share, run)[:m]
    w, h = (np.where(big, rng.integers(1, 40 * 32, m), rng.integers(1, 64, m)) / 32
            for _ in range(2))
    x, y = (rng.integers(-64, 64 * (n + 1), m) / 64 for _ in range(2))
    x, y, w, h = (np.asarray(a, np.float32) for a in (x, y, w, h))
    inst = dataclasses.replace(inst, x=x, y=y, w=w, h=h, xl=0.0, yl=0.0, bin_w=1.0, bin_h=1.0)
    ex, ey = (rng.standard_normal((n, n)).astype(np.float32) for _ in range(2))
    c = DeviceCells(inst)
    gx, gy = torch.full((m,), 7.0, device="cuda"), torch.full((m,), -3.0, device="cuda")
    dx, dy = (torch.as_tensor(v.ravel()).cuda() for v in (ex, ey))
    say("gather of large cells", m, n, share, run)
    for accumulate in (0, 1):
        F.field_gather(F.Grid.of(inst), c.x, c.y, c.w, c.h, dx, dy, None, "field", 0.5,
                       accumulate, gx, gy)
    torch.cuda.synchronize()
    rx, ry = oracle.field_gradient(inst, ex.astype(np.float64), ey.astype(np.float64))
    assert rel_l2(host(gx), rx) < RTOL and rel_l2(host(gy), ry) < RTOL
    # the small cells by themselves: the large ones would hide them in the norm
    assert rel_l2(host(gx)[~big], rx[~big]) < RTOL and rel_l2(host(gy)[~big], ry[~big]) < RTOL


# compact evaluations by form, most of them with the positions spread to the pins: grids
# of up to 256, with the row transform fused into the scatter and not, and past n =
# 512; the cells over the region, clustered, and crowded into a few bands
@pytest.mark.parametrize("where", ["uniform", "cluster", "crowd"])
@pytest.mark.parametrize("m,n,mode,dct", [
    (262145, 256, "field", "fft"), (300000, 128, "exact", "fft"), (300000, 64, "field", "fft"),
    (300000, 32, "exact", "fft"), (270001, 192, "field", "gemm_f32"),
    (300000, 512, "exact", "fft"), (300000, 1024, "field", "fft"),
    (300000, 576, "exact", "gemm_f32"),
    # cells of many bins each: the first designs of their grids in the compact form, and
    # the last on the general path
    (8192, 1024, "field", "fft"), (8191, 1024, "exact", "fft"), (2592, 576, "field", "gemm_f32"),
    (2591, 576, "exact", "gemm_f32")])
def test_eval_compact_forms(F, m, n, mode, dct, where):
    import torch
    inst = gen.make_instance((115, m, n), num_cells=m, util=0.8, n=n, num_nets=m, num_macros=2,
                             macro_area_frac=0.1, hi_frac=0.002, hi_range=(20, 400))
    if where != "uniform":
        rng, s = np.random.default_rng((116, m)), 0.15 if where == "cluster" else 0.01
        x, y = (np.clip(0.5 + s * rng.standard_normal(m), 0.01, 0.99) for _ in range(2))
        inst = dataclasses.replace(inst, x=(inst.xl + x * n * inst.bin_w).astype(np.float32),
                                   y=(inst.yl + y * n * inst.bin_h).astype(np.float32))
    plan, prob, c = F.Plan(n, dct), F.Problem.from_instance(inst), DeviceCells(inst)
    gx, gy = (torch.empty(m, device="cuda") for _ in range(2))
    out = torch.empty(4, dtype=torch.float64, device="cuda")
    say("eval", m, n, mode, dct, where)
    F.eval(plan, prob, c.x, c.y, 1.5, inst.gamma, mode, gx, gy, out)
    torch.cuda.synchronize()
    want = oracle.evaluate(inst, lam=1.5, grad_mode=mode)
    assert rel_l2(host(plan.maps()[0]), want["rho"]) < RTOL
    assert rel_l2(host(gx), want["gx"]) < RTOL and rel_l2(host(gy), want["gy"]) < RTOL
    o = host(out)
    for k, name in enumerate(("energy", "wa", "hpwl")):
        assert abs(o[k] - want[name]) <= RTOL * abs(want[name])
    assert abs(o[3] - want["overflow"]) < RTOL
    plan.close()


# a batch with a design past the compact form's cells among smaller ones is one group
# still: request i's maps in slot i, every result that of its own evaluation
@pytest.mark.parametrize("sizes,n,mode", [([3000, 1048577, 40000], 256, "field"),
                                          ([1048577, 300000, 5000], 1024, "exact")])
def test_batch_with_a_design_past_the_compact_form(F, sizes, n, mode):
    import torch
    insts = [gen.make_instance((117, k), num_cells=m, util=0.7, n=n, num_nets=m)
             for k, m in enumerate(sizes)]
    probs = [F.Problem.from_instance(i) for i in insts]
    cells = [DeviceCells(i) for i in insts]
    plan, single = F.Plan(n, max_batch=4), F.Plan(n)
    gxs, gys = ([torch.empty(m, device="cuda") for m in sizes] for _ in range(2))
    out = torch.empty((len(sizes), 4), dtype=torch.float64, device="cuda")
    say("batch", sizes, n, mode)
    F.eval_batch(plan, probs, [c.x for c in cells], [c.y for c in cells], [2.0] * len(sizes),
                 [i.gamma for i in insts], mode, gxs, gys, out)
    for k, i in enumerate(insts):
        gx, gy = (torch.empty(i.num_cells, device="cuda") for _ in range(2))
        o4 = torch.empty(4, dtype=torch.float64, device="cuda")
        F.eval(single, probs[k], cells[k].x, cells[k].y, 2.0, i.gamma, mode, gx, gy, o4)
        torch.cuda.synchronize()
        assert torch.equal(gx, gxs[k]) and torch.equal(gy, gys[k])
        assert torch.allclose(o4, out[k], rtol=1e-12, atol=0.0)
        assert torch.equal(single.maps()[0], plan.maps(k)[0])
    plan.close()
    single.close()


# many pins: more than 16384 in each block of cells, and more than 2,097,152 in all,
# which are handed their cells' positions up to 262,144 cells too
@pytest.mark.parametrize("m,n,nets,hi", [(300, 16, 14000, 8), (2000, 64, 60000, 8),
                                         (8193, 64, 720000, 8), (8192, 64, 720000, 8),
                                         (100000, 256, 700000, 3000)])
def test_eval_with_many_pins(F, m, n, nets, hi):
    import torch
    inst = gen.make_instance((118, m, nets), num_cells=m, util=0.7, n=n, num_nets=nets,
                             hi_frac=0.0002 if hi > 8 else 0.0, hi_range=(hi, hi))
    plan, prob, c = F.Plan(n), F.Problem.from_instance(inst), DeviceCells(inst)
    gx, gy, wx, wy = (torch.empty(m, device="cuda") for _ in range(4))
    out = torch.empty(4, dtype=torch.float64, device="cuda")
    wl, hp = (torch.empty(1, dtype=torch.float64, device="cuda") for _ in range(2))
    say("eval", m, n, inst.num_pins)
    F.eval(plan, prob, c.x, c.y, 1.5, inst.gamma, "field", gx, gy, out)
    F.problem_wl_grad(prob, c.x, c.y, inst.gamma, 0, wx, wy, wl, hp)
    torch.cuda.synchronize()
    want = oracle.evaluate(inst, lam=1.5, grad_mode="field")
    assert rel_l2(host(gx), want["gx"]) < RTOL and rel_l2(host(gy), want["gy"]) < RTOL
    for got, name in ((out[0], "energy"), (out[1], "wa"), (out[2], "hpwl"), (wl, "wa"),
                      (hp, "hpwl")):
        assert abs(float(got) - want[name]) <= RTOL * abs(want[name])
    W, rx, ry = oracle.wa_wirelength(inst)
    assert rel_l2(host(wx), rx) < RTOL and rel_l2(host(wy), ry) < RTOL
    plan.close()


# tall cells, past four bands high, in lists longer than a window of any block
@pytest.mark.parametrize("m,n,share", [(30000, 256, 0.1), (60000, 512, 0.06),
                                       (60000, 1024, 0.01)])
def test_many_tall_cells(F, m, n, share):
    import torch
    inst = gen.make_instance((119, m, n), num_cells=m, util=0.7, n=n, num_nets=m)
    h = inst.h.copy()
    k = np.random.default_rng((120, m)).random(m) < share
    h[k] = (24 * inst.bin_h) if n < 1024 else 40 * inst.bin_h
    inst = dataclasses.replace(inst, h=h)
    plan, prob, c = F.Plan(n), F.Problem.from_instance(inst), DeviceCells(inst)
    gx, gy = (torch.empty(m, device="cuda") for _ in range(2))
    out = torch.empty(4, dtype=torch.float64, device="cuda")
    rho = torch.empty(n * n, device="cuda")
    say("tall cells", m, n, int(k.sum()))
    F.problem_density(prob, c.x, c.y, rho)
    F.eval(plan, prob, c.x, c.y, 1.5, inst.gamma, "field", gx, gy, out)
    torch.cuda.synchronize()
    want = oracle.evaluate(inst, lam=1.5, grad_mode="field")
    assert rel_l2(host(rho).reshape(n, n), want["rho"]) < RTOL
    assert torch.equal(plan.maps()[0].reshape(-1), rho)
    assert rel_l2(host(gx), want["gx"]) < RTOL and rel_l2(host(gy), want["gy"]) < RTOL
    plan.close()
