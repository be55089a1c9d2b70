"""The wall terms beyond the strips of the whole-tile reverse step, against the
oracle (normwise 1e-12, the bar of every reverse variant): reflecting walls in x
(k_adj_wall) with their columns overlapping, in one tile and in two, and the row
whose ghost beyond a wall in y is past its tile's strip; and the step's time next
to walls in x."""
import numpy as np
import pytest
import torch

import oracle
from paper_1010_4124_amd import inputs, lbm

pytestmark = pytest.mark.gpu
P, F, R = 0, 1, 2
SIDES = [(1.1, 0.05, 0.0, 0.9), (0.8, -0.05, 0.02, 1.05), (1.0, 0.0, 0.05, 1.0),
         (0.9, 0.1, -0.05, 0.85)]
SHAPES = [(3, 6), (4, 3), (5, 10), (6, 9), (7, 14), (63, 22), (64, 6), (65, 7), (66, 10),
          (67, 18), (69, 4), (130, 26)]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    torch.cuda.set_device(0)


@pytest.mark.parametrize("bc", [(R, R, R, R), (R, F, P, P), (F, R, R, R), (R, R, F, R),
                                (R, R, P, P), (P, P, F, R)])
def test_parity(bc):
    for nx, ny in SHAPES:
        p = oracle.OracleParams.make(nx, ny, 2e-2, 2.5e-2, 4e-4, 6e-4, bc, side_state=SIDES)
        f = inputs.random_f(nx, ny, seed=nx + ny)
        lam = inputs.random_like(f.shape, seed=ny)
        ref = oracle.adjoint_step(p, f, lam, 0.7)
        ctx = lbm.Context(nx, ny, 2e-2, 2.5e-2, 4e-4, 6e-4, bc, side_state=SIDES)
        assert lbm.lbm_adjoint_variant_info(ctx.adj_variant) == (4, 18, 3, 0)
        got = ctx.adjoint_step(torch.from_numpy(f).cuda(), torch.from_numpy(lam).cuda(), 0.7)
        err = float(np.abs(got.cpu().numpy() - ref).max() / np.abs(ref).max())
        assert err < 1e-12, (nx, ny, bc, err)


@pytest.mark.parametrize("shape", [(64, 64), (64, 206), (128, 64), (500, 60)])
def test_default_is_not_slowed_by_walls_in_x(shape):
    """Against one workgroup per tile and velocity, the default of small boxes
    before the whole-tile kernel (which took 1.3 to 2.7 times its time here)."""
    info = [lbm.lbm_adjoint_variant_info(v) for v in range(lbm.lbm_adjoint_variant_count())]
    ctx = lbm.Context(*shape, 1e-3, 1e-3, 1e-5, 1e-5, (R, R, R, R))
    f = torch.from_numpy(inputs.random_f(*shape, seed=1)).cuda()
    lam, out = torch.randn_like(f), torch.empty_like(f)
    ms = []
    for v in (ctx.adj_variant, info.index((4, 18, 2, 1))):
        ctx.adj_variant = v
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        for n in (20, 200):
            e[0].record()
            for _ in range(n):
                ctx.adjoint_step(f, lam, 0.7, out=out)
            e[1].record()
            e[1].synchronize()
        ms.append(e[0].elapsed_time(e[1]))
    assert ms[0] < 1.15 * ms[1], ms
