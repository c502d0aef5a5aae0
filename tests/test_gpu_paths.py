"""The compact evaluation against the general exchange path on the same design, and
the general path where the compact form ends.  A problem that declares nets of up to
3900 pins has net blocks too large for the compact form, whatever its nets are."""
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


def _run(F, inst, mode, dct, max_degree, wl):
    import torch
    prob = F.Problem(F.Grid.of(inst), *(dev(getattr(inst, k)) for k in
                                        ("w", "h", "net_ptr", "pin_cell", "pin_dx", "pin_dy")),
                     max_degree=max_degree, wl_model=wl)
    plan, c = F.Plan(inst.n, dct), DeviceCells(inst)
    gx, gy = (torch.empty(inst.num_cells, device="cuda") for _ in range(2))
    out, only = (torch.empty(4, dtype=torch.float64, device="cuda") for _ in range(2))
    F.eval(plan, prob, c.x, c.y, 1.5, inst.gamma, mode, gx, gy, out)
    F.eval(plan, prob, c.x, c.y, 1.5, inst.gamma, mode, None, None, only)
    torch.cuda.synchronize()
    rho = plan.maps()[0].clone()
    plan.close()
    return rho, gx, gy, out, only


# the same products in the same order on both paths: maps and gradients bit for bit, the
# totals up to the order of their double-precision partial sums (at most 2^16 of them,
# half an ulp each: 1e-11)
@pytest.mark.parametrize("m,n,mode,dct,wl", [
    (2000, 64, "field", "fft", "wa"), (8192, 16, "exact", "fft", "wa"),
    (30011, 256, "exact", "fft", "lse"), (9000, 192, "field", "gemm_f32", "wa"),
    (200000, 512, "field", "fft", "wa"), (60000, 1024, "exact", "fft", "wa"),
    (270001, 128, "field", "fft", "wa"), (300000, 1024, "field", "fft", "wa"),
    (530000, 512, "exact", "fft", "wa")])
def test_compact_equals_general(F, m, n, mode, dct, wl):
    import torch
    inst = gen.make_instance((130, m, n), num_cells=m, util=0.8, n=n, num_nets=m, hi_frac=0.002,
                             hi_range=(20, 400))
    say("compact and general", m, n, mode, dct, wl)
    most = int(np.diff(inst.net_ptr).max())
    assert most <= 400
    a, b = (_run(F, inst, mode, dct, d, wl) for d in (most, 3900))
    for p, q in zip(a[:3], b[:3]):
        assert torch.equal(p, q)
    for p, q in zip(a[3:], b[3:]):
        assert torch.allclose(p, q, rtol=1e-11, atol=0.0)
    assert torch.allclose(a[3], a[4], rtol=1e-11, atol=0.0)


@pytest.mark.parametrize("mode", ["field", "exact"])
def test_general_past_the_compact_cells(F, mode):
    inst = gen.make_instance(131, num_cells=1048577, util=0.8, n=512, num_nets=1060000)
    say("general", inst.num_cells, mode)
    rho, gx, gy, out, only = _run(F, inst, mode, "fft", int(np.diff(inst.net_ptr).max()), "wa")
    ref = oracle.evaluate(inst, lam=1.5, grad_mode=mode)
    assert rel_l2(host(rho), ref["rho"]) < RTOL
    assert rel_l2(host(gx), ref["gx"]) < RTOL and rel_l2(host(gy), ref["gy"]) < RTOL
    for o in (host(out), host(only)):
        for k, name in enumerate(("energy", "wa", "hpwl")):
            assert abs(o[k] - ref[name]) <= RTOL * abs(ref[name])
