"""The size rules of the launches: designs at the edges where the blocks of a
kernel change their size, against the FP64 oracle (relative L2 <= 1e-5, the
bar of every float32 result here)."""
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


# cells per counting block 512 | 1024 | 2048 | 4096, the band kernels' small and
# large forms (n <= 512 and up to 1024 cells per band), odd and tiny grids
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
