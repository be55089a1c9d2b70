"""The upwind schemes' kernel of one thread per cell, which tall grids of a few
columns take, against the oracle (normwise 1e-12, the bar of the schemes' other
cases): every boundary kind on both axes, ragged 256-cell blocks, one column."""
import numpy as np
import pytest
import torch

import oracle
from paper_1010_4124_amd import inputs, lbm

pytestmark = pytest.mark.gpu
P, F, R, O = 0, 1, 2, 3
SIDES = [(1.1, 0.05, 0.0, 0.9), (0.8, -0.05, 0.02, 1.05), (1.0, 0.0, 0.05, 1.0),
         (0.9, 0.1, -0.05, 0.85)]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    torch.cuda.set_device(0)


@pytest.mark.parametrize("nx,ny,bc", [(1, 16001, (P, P, R, R)), (3, 16003, (R, F, P, P)),
                                      (4, 20001, (F, R, O, F)), (5, 20002, (O, O, R, O)),
                                      (4, 17000, (P, P, P, P))])
@pytest.mark.parametrize("scheme", [lbm.UPWIND1, lbm.UPWIND2])
def test_parity(nx, ny, bc, scheme):
    assert lbm.lib().lbmi_upwind_rows(scheme, nx, ny) == 0
    f = inputs.random_f(nx, ny, seed=ny)
    p = oracle.OracleParams.make(nx, ny, 2e-2, 2.5e-2, 4e-4, 6e-4, bc, side_state=SIDES,
                                 scheme=scheme)
    want = oracle.step(p, f, 3, nthreads=8)
    ctx = lbm.Context(nx, ny, 2e-2, 2.5e-2, 4e-4, 6e-4, bc, side_state=SIDES, scheme=scheme)
    got, ke = ctx.step(torch.from_numpy(f).cuda(), 3, ke_log=True)
    assert np.abs(got.cpu().numpy() - want).max() <= 1e-12 * np.abs(want).max()
    assert ke[0].cpu().numpy() == pytest.approx(np.asarray(oracle.kinetic_y(p, f)), rel=1e-12)
