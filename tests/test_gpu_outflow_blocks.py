"""Outflow ghosts by workgroups of 64 positions: sides around one and two of them
against the oracle (normwise 1e-12, the bar of the step's other cases), alone and
in a batch, and the step's time next to long outflow sides in x."""
import numpy as np
import pytest
import torch

import oracle
from paper_1010_4124_amd import inputs, lbm

pytestmark = pytest.mark.gpu
P, F, R, O = 0, 1, 2, 3
CELL = (2e-2, 2.5e-2, 4e-4, 6e-4)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    torch.cuda.set_device(0)


@pytest.mark.parametrize("bc", [(O, O, P, P), (P, P, O, O), (O, O, O, O)])
def test_parity(bc):
    shapes = [(63, 65), (64, 64), (65, 63), (5, 129), (128, 3), (200, 127)]
    b = lbm.Batch([lbm.LbmParams.make(nx, ny, *CELL, bc) for nx, ny in shapes])
    f = [inputs.random_f(nx, ny, seed=nx) for nx, ny in shapes]
    out = b.step(torch.cat([torch.from_numpy(q).reshape(-1) for q in f]).cuda(), 3)
    for i, (nx, ny) in enumerate(shapes):
        want = oracle.step(oracle.OracleParams.make(nx, ny, *CELL, bc), f[i], 3)
        got = lbm.Context(nx, ny, *CELL, bc).step(torch.from_numpy(f[i]).cuda(), 3)
        for g in (got, b.view(out, i)):
            assert np.abs(g.cpu().numpy() - want).max() <= 1e-12 * np.abs(want).max(), (nx, ny)


def test_default_is_not_slowed_by_outflow_in_x():
    """Against the state pass and plane kernel, which write the ghosts themselves
    and were the default of such grids before the whole-tile step."""
    info = [lbm.lbm_step_variant_info(v) for v in range(lbm.lbm_step_variant_count())]
    ctx = lbm.Context(320, 250, *CELL, (O, O, P, P))
    f = torch.from_numpy(inputs.random_f(320, 250, seed=1)).cuda()
    out, ms = torch.empty_like(f), []
    for v in (ctx.variant, info.index((4, 18, 4, 1, 0, 2))):
        ctx.variant = v
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        for n in (50, 400):
            e[0].record()
            ctx.step(f, n, out=out)
            e[1].record()
            e[1].synchronize()
        ms.append(e[0].elapsed_time(e[1]))
    assert ms[0] < 1.05 * ms[1], ms
