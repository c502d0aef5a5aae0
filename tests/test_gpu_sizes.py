"""The size rules of the launches: designs at the edges where the blocks of a
kernel change their size, against the FP64 oracle (relative L2 <= 1e-5, the
bar of every float32 result here)."""
import dataclasses

import numpy as np
import pytest

import gen
import oracle
from _helpers import rel_l2
from gpu_common import RTOL, DeviceCells, dev, host, lib_or_build, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    lib_or_build()
    from paper_1312_4587_amd import fftpl
    return fftpl


# cells per counting block 512 | 1024 | 2048 | 4096, bands of one row (up to n = 256)
# to four, odd and tiny grids
@pytest.mark.parametrize("m,n", [(1, 8), (511, 1), (513, 3), (2000, 100), (131072, 256),
                                 (131073, 512), (131073, 513), (262145, 512), (262145, 300),
                                 (524289, 512), (524289, 1024), (1048577, 1000)])
def test_density_map_block_sizes(F, m, n):
    import torch
    inst = gen.make_instance((92, m, n), num_cells=m, util=0.7, n=n, num_nets=1 if m > 9 else 0,
                             num_macros=2, macro_area_frac=0.1)
    grid = F.Grid.of(inst)
    c = DeviceCells(inst)
    b0, _ = oracle.fixed_maps(inst)
    base = torch.as_tensor(np.asarray(b0, np.float32).ravel()).cuda()
    rho = torch.empty(n * n, device="cuda")
    say("density", m, n)
    F.density_map(grid, c.x, c.y, c.w, c.h, base, rho)
    torch.cuda.synchronize()
    assert rel_l2(host(rho).reshape(n, n), oracle.density_map(inst, b0)) < RTOL


# small maps in one launch, without band lists (up to 16384 cells with n <= 256, 8192
# with n <= 512), and the first designs past it; no cells; each into an old map and again
@pytest.mark.parametrize("m,n", [(0, 16), (1, 1), (2047, 31), (2049, 64), (8192, 512),
                                 (8193, 512), (8192, 513), (5000, 7), (16384, 128), (16385, 128)])
def test_density_map_small(F, m, n):
    import torch
    inst = gen.make_instance((100, m, n), num_cells=max(m, 1), util=0.7, n=n, num_nets=0,
                             num_macros=2, macro_area_frac=0.1)
    inst = dataclasses.replace(inst, **{k: getattr(inst, k)[:m] for k in "xywh"})
    c = DeviceCells(inst)
    b0, _ = oracle.fixed_maps(inst)
    base = torch.as_tensor(np.asarray(b0, np.float32).ravel()).cuda()
    rho = torch.full((n * n,), 7.0, device="cuda")
    want = oracle.density_map(inst, b0) if m else np.asarray(b0)
    say("density", m, n)
    for b, ref in ((base, want), (None, want - b0)):
        F.density_map(F.Grid.of(inst), c.x, c.y, c.w, c.h, b, rho)
        torch.cuda.synchronize()
        # (m = 0 without a base is the zero map)
        assert rel_l2(host(rho).reshape(n, n), ref) < RTOL or not (ref.any() or host(rho).any())


def _eval(F, inst, mode, dct="fft", shift=0, **prob_kw):
    """One evaluation with the positions `shift` floats into a larger array."""
    import torch
    prob = F.Problem.from_instance(inst, **prob_kw)
    plan = F.Plan(inst.n, dct)
    m = inst.num_cells
    x, y, gx, gy = (torch.zeros(m + shift, device="cuda")[shift:] for _ in range(4))
    x.copy_(torch.as_tensor(inst.x))
    y.copy_(torch.as_tensor(inst.y))
    out = torch.empty(4, dtype=torch.float64, device="cuda")
    F.eval(plan, prob, x, y, 1.5, inst.gamma, mode, gx, gy, out)
    only = torch.empty(4, dtype=torch.float64, device="cuda")
    F.eval(plan, prob, x, y, 1.5, inst.gamma, mode, None, None, only)
    torch.cuda.synchronize()
    got = dict(gx=host(gx), gy=host(gy), out=host(out), only=host(only),
               rho=host(plan.maps()[0]))
    plan.close()
    return got


def _check(inst, got, mode, **kw):
    ref = oracle.evaluate(inst, lam=1.5, grad_mode=mode, **kw)
    assert rel_l2(got["rho"], ref["rho"]) < RTOL
    assert rel_l2(got["gx"], ref["gx"]) < RTOL and rel_l2(got["gy"], ref["gy"]) < RTOL
    for o in (got["out"], got["only"]):
        for k, name in enumerate(("energy", "wa", "hpwl")):
            assert abs(o[k] - ref[name]) <= RTOL * abs(ref[name])
        assert abs(o[3] - ref["overflow"]) < RTOL


# the compact evaluation's forms: cells read by every band block up to 8192,
# then a place pass; row transforms fused from n = 64; cell blocks of 256 to 2048
# cells (524,288 cells) and of 4096; positions read by pin up to 262,144 cells
@pytest.mark.parametrize("m,n,mode", [
    (1, 8, "field"), (257, 16, "exact"), (1000, 32, "field"), (4097, 64, "field"),
    (8192, 128, "exact"), (8193, 128, "field"), (40000, 256, "exact"), (131073, 512, "field"),
    (262145, 512, "field"), (524288, 512, "exact"), (524289, 512, "field"),
    (300000, 1024, "field")])
def test_eval_sizes(F, m, n, mode):
    inst = gen.make_instance((93, m, n), num_cells=m, util=0.7, n=n,
                             num_nets=int(1.1 * m) if m > 9 else 0, num_macros=3,
                             macro_area_frac=0.1)
    say("eval", m, n, mode)
    _check(inst, _eval(F, inst, mode, shift=1), mode)


# compact evaluations past n = 512 (bands of three and four rows, the row pass on
# its own), with the positions read by pin up to 262,144 cells and spread past them;
# the matrix-core solve among them; cells of several bins each way, and one cell on
# n = 1024, which is left to the general path
@pytest.mark.parametrize("m,n,mode,dct", [
    (1, 1024, "field", "fft"), (8192, 1024, "exact", "fft"), (30000, 640, "field", "gemm_f32"),
    (262144, 1024, "exact", "fft"), (262145, 1024, "field", "fft"), (262145, 576, "exact", "gemm_f32"),
    (270000, 1024, "field", "gemm_bf16x3"), (524288, 1024, "exact", "fft"),
    (524289, 1024, "field", "fft"), (20, 8, "field", "fft"), (20, 64, "exact", "fft")])
def test_eval_large_grids(F, m, n, mode, dct):
    inst = gen.make_instance((97, m, n), num_cells=m, util=0.8, n=n,
                             num_nets=int(1.05 * m) if m > 9 else 0, num_macros=2,
                             macro_area_frac=0.1, hi_frac=0.002 if m > 20000 else 0.0,
                             hi_range=(20, 400))
    say("eval", m, n, mode, dct)
    _check(inst, _eval(F, inst, mode, dct=dct), mode)


# cell blocks of up to 4096 cells (1,048,576 cells, place blocks of 4096 too), and
# the general path past them
@pytest.mark.parametrize("m,n,mode,dct", [
    (600001, 1024, "exact", "fft"), (524289, 512, "exact", "fft"),
    (1048576, 1024, "field", "fft"), (1048577, 1024, "exact", "fft"),
    (1000000, 704, "field", "gemm_f32")])
def test_eval_million_cells(F, m, n, mode, dct):
    inst = gen.make_instance((101, m, n), num_cells=m, util=0.8, n=n, num_nets=int(1.02 * m),
                             num_macros=2, macro_area_frac=0.1, hi_frac=0.001,
                             hi_range=(20, 400))
    say("eval", m, n, mode, dct)
    _check(inst, _eval(F, inst, mode, dct=dct), mode)


def test_batch_spreads_together(F):
    # designs whose positions are spread to the pins beside ones read by the band
    # blocks, placed first, and on the general path
    import torch
    sizes = [(3000, 0), (270000, 0), (30000, 0), (20000, 4800)]
    insts = [gen.make_instance((98, k), num_cells=m, util=0.7, n=1024, num_nets=m,
                               hi_frac=0.001 if d else 0.0, hi_range=(d, d))
             for k, (m, d) in enumerate(sizes)]
    probs = [F.Problem.from_instance(i) for i in insts]
    cells = [DeviceCells(i) for i in insts]
    plan, single = F.Plan(1024, max_batch=4), F.Plan(1024)
    gxs, gys = ([torch.empty(i.num_cells, device="cuda") for i in insts] for _ in range(2))
    out = torch.empty((len(insts), 4), dtype=torch.float64, device="cuda")
    say("batch with a spread")
    F.eval_batch(plan, probs, [c.x for c in cells], [c.y for c in cells], [2.0] * len(insts),
                 [i.gamma for i in insts], "exact", gxs, gys, out)
    for k, i in enumerate(insts):
        gx, gy = (torch.empty(i.num_cells, device="cuda") for _ in range(2))
        o4 = torch.empty(4, dtype=torch.float64, device="cuda")
        F.eval(single, probs[k], cells[k].x, cells[k].y, 2.0, i.gamma, "exact", gx, gy, o4)
        torch.cuda.synchronize()
        assert torch.equal(gx, gxs[k]) and torch.equal(gy, gys[k])
        assert torch.allclose(o4, out[k], rtol=1e-12, atol=0.0)
    plan.close()
    single.close()


# net blocks at their size rules: one staging round, several, the largest that
# two share a CU, and past it (the general path); pins above 2,048 per block
@pytest.mark.parametrize("hi", [900, 1100, 3000, 4700])
def test_eval_net_block_sizes(F, hi):
    inst = gen.make_instance((94, hi), num_cells=20000, util=0.7, n=128, num_nets=21000,
                             hi_frac=0.003, hi_range=(hi, hi))
    say("eval, nets of", hi)
    for wl in ("wa", "lse"):
        _check(inst, _eval(F, inst, "field", wl_model=wl), "field", wl_model=wl)


def test_eval_sizes_with_matrix_cores(F):
    # scatter and net blocks in one launch, the solve on the matrix cores
    for m, n in ((9000, 192), (5000, 128)):
        inst = gen.make_instance((95, m), num_cells=m, util=0.7, n=n, num_nets=m)
        for mode in ("field", "exact"):
            say("eval gemm_f32", m, n, mode)
            _check(inst, _eval(F, inst, mode, dct="gemm_f32"), mode)


def test_batch_mixes_size_classes(F):
    # one call with designs read by the band blocks, placed first, and on the
    # general path (nets too large for the compact form): each equals its own
    # single evaluation
    import torch
    sizes = [(3000, 8), (8192, 8), (8193, 8), (15000, 4800), (12000, 8)]
    insts = [gen.make_instance((96, k), num_cells=m, util=0.7, n=128, num_nets=m,
                               hi_frac=0.001 if d > 8 else 0.0, hi_range=(d, d))
             for k, (m, d) in enumerate(sizes)]
    probs = [F.Problem.from_instance(i) for i in insts]
    cells = [DeviceCells(i) for i in insts]
    plan, single = F.Plan(128, max_batch=8), F.Plan(128)
    gxs, gys = ([torch.empty(i.num_cells, device="cuda") for i in insts] for _ in range(2))
    out = torch.empty((len(insts), 4), dtype=torch.float64, device="cuda")
    F.eval_batch(plan, probs, [c.x for c in cells], [c.y for c in cells], [2.0] * len(insts),
                 [i.gamma for i in insts], "field", gxs, gys, out)
    for k, i in enumerate(insts):
        gx, gy = (torch.empty(i.num_cells, device="cuda") for _ in range(2))
        o4 = torch.empty(4, dtype=torch.float64, device="cuda")
        F.eval(single, probs[k], cells[k].x, cells[k].y, 2.0, i.gamma, "field", gx, gy, o4)
        torch.cuda.synchronize()
        assert torch.equal(gx, gxs[k]) and torch.equal(gy, gys[k])
        assert torch.allclose(o4, out[k], rtol=1e-12, atol=0.0)
    plan.close()
    single.close()


# the stateless wirelength gradient: lane pairs up to degree 8, a wavefront from
# 9 (registers up to 1,024 pins, several passes past them), one launch for both;
# net and cell counts around its blocks; accumulating, the totals left out, and a
# non-finite position, which makes its nets' cells NaN and no other cell
@pytest.mark.parametrize("m,degs", [(1, [1, 1]), (70, [8] * 127 + [9]), (127, [2] * 129),
                                    (300, [64, 65, 0, 1, 63, 2, 3]),
                                    (3000, [1024, 1025, 2, 2100, 8, 9] + [5] * 300)])
def test_stateless_wirelength_sizes(F, m, degs):
    import torch
    base = gen.make_instance((97, m), num_cells=m, util=0.7, n=16, num_nets=0)
    rng = np.random.default_rng(97)
    cells = np.concatenate([rng.choice(m, size=d, replace=False) for d in degs]).astype(np.int32)
    inst = dataclasses.replace(
        base, net_ptr=np.concatenate([[0], np.cumsum(degs)]).astype(np.int32), pin_cell=cells,
        pin_dx=(rng.random(len(cells)) - 0.5).astype(np.float32),
        pin_dy=(rng.random(len(cells)) - 0.5).astype(np.float32))
    c = DeviceCells(inst)
    net = (dev(inst.net_ptr), dev(inst.pin_cell), dev(inst.pin_dx), dev(inst.pin_dy))
    for call, ref in ((F.wa_grad, oracle.wa_wirelength), (F.lse_grad, oracle.lse_wirelength)):
        gx, gy = (torch.full((m,), 3.0, device="cuda") for _ in range(2))
        wl, hp = (torch.zeros(1, dtype=torch.float64, device="cuda") for _ in range(2))
        say("stateless", m, len(degs), call.__name__)
        call(*net, c.x, c.y, inst.gamma, 0, gx, gy, wl, hp)
        W0, rx, ry = ref(inst)
        scale = max(1.0, np.linalg.norm(rx), np.linalg.norm(ry))
        assert np.linalg.norm(host(gx) - rx) < RTOL * scale
        assert np.linalg.norm(host(gy) - ry) < RTOL * scale
        assert abs(float(wl) - W0) <= RTOL * max(abs(W0), inst.gamma)
        assert abs(float(hp) - oracle.hpwl(inst)) <= RTOL * oracle.hpwl(inst)
        ax, ay = gx.clone(), gy.clone()
        call(*net, c.x, c.y, inst.gamma, 1, ax, ay)
        torch.cuda.synchronize()
        assert torch.equal(ax, gx + gx) and torch.equal(ay, gy + gy)
    bad = int(cells[-1])
    x = c.x.clone()
    x[bad] = float("nan")
    F.wa_grad(*net, x, c.y, inst.gamma, 0, ax, ay)
    deg = np.diff(inst.net_ptr)
    net_of = np.repeat(np.arange(len(deg)), deg)
    hit = np.zeros(m, bool)
    for e in np.unique(net_of[cells == bad]):
        if deg[e] >= 2:
            hit[cells[net_of == e]] = True
    assert np.array_equal(np.isnan(host(ax)), hit)


# the standalone gather's fast forms (a row's bins in one or two loads: four columns of
# two rows, eight of three) and its loops, grids too narrow for the wide loads, and
# one map after the other from 524288 cells at n >= 1024
@pytest.mark.parametrize("mode", ["field", "exact"])
@pytest.mark.parametrize("m,n", [(1, 1), (300, 3), (300, 4), (2000, 37), (524287, 1024),
                                 (524288, 1024), (524545, 1030)])
def test_field_gather_sizes(F, mode, m, n):
    import torch
    inst = gen.make_instance((94, m, n), num_cells=m, util=0.7, n=n, num_nets=0)
    rng = np.random.default_rng((95, m, n))
    # unit bins and dyadic edges, so that float32 and the oracle see the same bins:
    # edges on and off bin edges, cells over and past the border, up to six bins
    w, h = (rng.integers(1, 75, m) / 32 for _ in range(2))
    x, y = (rng.integers(0, 64 * n, m) / 64 for _ in range(2))
    k = min(m, 4000)
    w[:k], h[:k] = rng.integers(1, 6, k), rng.integers(1, 6, k)
    x[:k] = rng.integers(-1, n + 2, k) + 0.5 * rng.integers(0, 2, k)
    y[:k] = rng.integers(-1, n + 2, k) + 0.5 * rng.integers(0, 2, k)
    x, y, w, h = (np.asarray(a, np.float32) for a in (x, y, w, h))
    inst = dataclasses.replace(inst, x=x, y=y, w=w, h=h, xl=0.0, yl=0.0, bin_w=1.0, bin_h=1.0)
    ex, ey, psi = (rng.standard_normal((n, n)).astype(np.float32) for _ in range(3))
    c = DeviceCells(inst)
    gx, gy = torch.full((m,), 7.0, device="cuda"), torch.full((m,), -3.0, device="cuda")
    say("gather", mode, m, n)
    for accumulate in (0, 1):
        F.field_gather(F.Grid.of(inst), c.x, c.y, c.w, c.h, dev(ex.ravel()), dev(ey.ravel()),
                       dev(psi.ravel()), mode, 0.5, accumulate, gx, gy)
    torch.cuda.synchronize()
    if mode == "field":
        rx, ry = oracle.field_gradient(inst, ex.astype(np.float64), ey.astype(np.float64))
    else:
        rx, ry = oracle.exact_gradient(inst, psi.astype(np.float64))
    assert rel_l2(host(gx), rx) < RTOL and rel_l2(host(gy), ry) < RTOL
